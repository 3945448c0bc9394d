// Learned combiner: a 16 -> 64 -> 64 -> 1 ReLU network in FP32 that maps the
// H = 16 per-hash lifted sizes of a node (log-scaled) to an estimate of its
// log out-component size.  Forward and backward run on the FP32 matrix
// instruction (16 x 16 x 4, FP32 in, FP32 sums); partial gradients of the
// workgroups are summed in a fixed order, so a training step is bit-for-bit
// deterministic.
//
// Parameter layout (5313 floats): W1 (64 x 16, row-major), b1 (64),
// W2 (64 x 64), b2 (64), W3 (1 x 64), b3 (1).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "tn_mlp.h"

namespace tn {

namespace {

constexpr int kIn = 16, kH = 64;
constexpr int oW1 = 0, oB1 = oW1 + kH * kIn, oW2 = oB1 + kH, oB2 = oW2 + kH * kH, oW3 = oB2 + kH,
              oB3 = oW3 + kH, kParams = oB3 + 1;
static_assert(kParams == 5313, "parameter count");

// Matrix tiles.  D (16 x 16) += A (16 x 4) B (4 x 16): lane l holds
// A[l % 16][l / 16], B[l / 16][l % 16] and D[4 (l / 16) + r][l % 16], r < 4.
// Samples are the columns of B and D, a layer's units the rows of A and D,
// and the order in which k runs over a layer's inputs is free as long as A
// and B agree.
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Four consecutive floats; one 16-byte load where `wide` (uniform) says that
// the array starts on 16 bytes (p is a multiple of 4 floats into it).
__device__ __forceinline__ f4 load4(const float *__restrict__ p, bool wide) {
    if (wide) return *(const f4 *)p;
    f4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = p[i];
    return v;
}

__device__ __forceinline__ bool on16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

// max(v, 0), and 0 for NaN, as fmaxf: the median with 0 and infinity, one
// instruction where fmaxf first quiets a NaN in one of its own.  (top() hides
// the infinity from the compiler, which would make it fmaxf again.)
__device__ __forceinline__ float top() {
    float v = __builtin_inff();
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ float relu(float v, float inf) {
    return __builtin_amdgcn_fmed3f(v, 0.f, inf);
}

__device__ __forceinline__ f4 relu4(f4 v, float inf) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = relu(v[i], inf);
    return v;
}

// Outputs of N samples: yhat, or with PREDICT n_nodes e^yhat clamped.
//
// A wavefront keeps every weight in registers (W1 16, W2 64, biases and W3
// 48 a lane) and takes tiles of 16 samples.  The hidden units of a tile
// leave the first layer as D tiles, lane l holding units 16 t + 4 (l / 16) +
// r of sample l % 16: exactly a B operand whose k runs over t and r, so the
// second layer reads them where they are, with W2 loaded in the same order.
// No LDS and no exchange but the output's sum over the four lane groups.
// Bound by the matrix cores (80 instructions of 32 cycles per tile, 67 us at
// N = 10^6; 83 % of the time that wavefronts run): 101 us (103 TFLOP/s), 112 us
// with rows that were only requested once the tile before was done and two
// instructions a ReLU, 302 us (34 TFLOP/s) with one sample per lane on the
// vector units, the weights broadcast from LDS.  Outputs a tile late, under the
// next one's products, or rows two tiles ahead, took the same 101 us.
template <bool PREDICT, bool WIDE, bool BOUND>
__global__ void __launch_bounds__(256)
k_mlp_outputs(const float *__restrict__ params, const float *__restrict__ x, int64_t N,
              uint32_t n_nodes, const int32_t *__restrict__ est, float *__restrict__ out) {
    const uint32_t lane = threadIdx.x & 63u, col = lane & 15u, g = lane >> 4;
    const int64_t tiles = (N + 15) / 16;
    const int64_t step = (int64_t)gridDim.x * (blockDim.x >> 6);
    int64_t tile = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const bool pwide = on16(params);
    f4 w1[4], w2[4][4], b1[4], b2[4], w3[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        w1[t] = load4(params + oW1 + (16 * t + col) * kIn + 4 * g, pwide);
        b1[t] = load4(params + oB1 + 16 * t + 4 * g, pwide);
        b2[t] = load4(params + oB2 + 16 * t + 4 * g, pwide);
        w3[t] = load4(params + oW3 + 16 * t + 4 * g, pwide);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            w2[t][k] = load4(params + oW2 + (16 * t + col) * kH + 16 * k + 4 * g, pwide);
    }
    const float b3 = params[oB3], inf = top();
    // a tile's rows, and what bounds its estimates (the last sample's past the
    // last one); unconditional, so that they stay in flight for a whole tile
    struct Rows {
        f4 x;
        int32_t most;
    };
    auto fetch = [&](int64_t tl) {
        const int64_t s = min(tl * 16 + col, N - 1);
        const float *p = x + s * kIn + 4 * g;
        Rows r;
        if constexpr (WIDE) {
            r.x = *(const f4 *)p;
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) r.x[q] = p[q];
        }
        r.most = PREDICT && BOUND ? est[s] : 0;
        return r;
    };
    Rows now = fetch(tile);
    for (; tile < tiles; tile += step) {
        const Rows next = fetch(tile + step);
        __builtin_amdgcn_sched_barrier(0);  // requested before this tile, not after it
        f4 h[4], z[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) h[t] = b1[t];
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int t = 0; t < 4; ++t) h[t] = mfma4(w1[t][k], now.x[k], h[t]);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            h[t] = relu4(h[t], inf);
            z[t] = b2[t];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int t = 0; t < 4; ++t) z[t] = mfma4(w2[t][k][r], h[k][r], z[t]);
        float y = 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) y = fmaf(w3[t][r], relu(z[t][r], inf), y);
        y += __shfl_xor(y, 16, 64);
        y += __shfl_xor(y, 32, 64);
        y += b3;
        const int64_t s = tile * 16 + col;
        if (g == 0 && s < N) {
            if (PREDICT) {
                const float hi = BOUND ? (float)now.most : (float)n_nodes;
                out[s] = fminf(fmaxf((float)n_nodes * expf(y), 1.f), hi);
            } else {
                out[s] = y;
            }
        }
        now = next;
    }
}

// Per-workgroup partial gradients of the mean squared error (scaled by 2/N)
// and its partial loss (sum of squared residuals / N).
//
// A workgroup of four wavefronts takes tiles of 32 samples; wavefront w owns
// units 16 w .. 16 w + 15 of either hidden layer (its rows of W1 and W2 and
// its columns of W2 in registers) for both halves of the tile.  Activations
// and deltas cross between the wavefronts through LDS, one row per sample;
// weight gradients are matrix products over the tile's samples, added up in
// registers over the workgroup's tiles.  At 4096 samples a step is latency:
// 128 workgroups run 9.2 us, where one sample per lane on 64 single
// wavefronts, each dot product of the weight gradients a serial chain, took
// 113 us.
constexpr int kTile = 32;
constexpr int kMaxPartials = 256;  // partial gradients of a step at most: one per CU
constexpr int kStride = kH + 4;    // LDS row: 16-byte aligned, rows on shifted banks
__global__ void __launch_bounds__(256)
k_mlp_backward(const float *__restrict__ params, const float *__restrict__ x,
               const float *__restrict__ y, const int32_t *__restrict__ idx, int64_t N,
               float *__restrict__ partial, float *__restrict__ loss_partial) {
    __shared__ __align__(16) float sx[kTile][kIn + 4];
    __shared__ __align__(16) float sh1[kTile][kStride];
    __shared__ __align__(16) float sd2[kTile][kStride];
    __shared__ __align__(16) float sd1[kTile][kStride];
    __shared__ float sy[4][kTile];
    const uint32_t lane = threadIdx.x & 63u, col = lane & 15u, g = lane >> 4;
    const uint32_t w = threadIdx.x >> 6, u0 = 16 * w + 4 * g;  // the lane's four units in D
    const bool pwide = on16(params), xwide = on16(x);
    const f4 w1 = load4(params + oW1 + (16 * w + col) * kIn + 4 * g, pwide);
    const f4 b1 = load4(params + oB1 + u0, pwide), b2 = load4(params + oB2 + u0, pwide);
    const f4 w3 = load4(params + oW3 + u0, pwide);
    const float b3 = params[oB3], inf = top();
    f4 w2[4], w2t[4];  // rows, and columns, of W2: k runs over 16 g + 4 q + r
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        w2[q] = load4(params + oW2 + (16 * w + col) * kH + 16 * g + 4 * q, pwide);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            w2t[q][r] = params[oW2 + (16 * g + 4 * q + r) * kH + 16 * w + col];
    }
    const float inv_n = 1.f / (float)N;
    f4 gw2[4] = {}, gw1 = {}, gb1 = {}, gb2 = {}, gw3 = {};
    float gb3 = 0.f, loss = 0.f;
    const int64_t tiles = (N + kTile - 1) / kTile;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        f4 h1[2], z2[2];
        float target[2];
        bool valid[2];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const int64_t s = tile * kTile + 16 * a + col;
            valid[a] = s < N;
            const int64_t row = valid[a] ? (idx ? (int64_t)idx[s] : s) : 0;
            const f4 xi = valid[a] ? load4(x + row * kIn + 4 * g, xwide) : f4{};
            target[a] = valid[a] ? y[row] : 0.f;
            if (w == 0) *(f4 *)&sx[16 * a + col][4 * g] = xi;
            h1[a] = b1;
#pragma unroll
            for (int k = 0; k < 4; ++k) h1[a] = mfma4(w1[k], xi[k], h1[a]);
        }
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            h1[a] = relu4(h1[a], inf);
            *(f4 *)&sh1[16 * a + col][u0] = h1[a];
        }
        __syncthreads();
#pragma unroll
        for (int a = 0; a < 2; ++a) z2[a] = b2;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            f4 hb[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) hb[a] = *(const f4 *)&sh1[16 * a + col][16 * g + 4 * q];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int a = 0; a < 2; ++a) z2[a] = mfma4(w2[q][r], hb[a][r], z2[a]);
        }
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            float v = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) v = fmaf(w3[r], fmaxf(z2[a][r], 0.f), v);
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if (g == 0) sy[w][16 * a + col] = v;
        }
        __syncthreads();
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const int c = 16 * a + col;
            const float out = ((sy[0][c] + sy[1][c]) + (sy[2][c] + sy[3][c])) + b3;
            const float res = valid[a] ? out - target[a] : 0.f;
            const float dy = 2.f * res * inv_n;
            gb3 += dy;
            loss = fmaf(res * inv_n, res, loss);
            f4 d2;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                d2[r] = z2[a][r] > 0.f ? dy * w3[r] : 0.f;
                gw3[r] = fmaf(dy, fmaxf(z2[a][r], 0.f), gw3[r]);
            }
            gb2 += d2;
            *(f4 *)&sd2[c][u0] = d2;
        }
        __syncthreads();
        // deltas of the first layer, and the gradient of W2's rows 16 w ..
        f4 d1[2] = {};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            f4 db[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) db[a] = *(const f4 *)&sd2[16 * a + col][16 * g + 4 * q];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int a = 0; a < 2; ++a) d1[a] = mfma4(w2t[q][r], db[a][r], d1[a]);
        }
#pragma unroll
        for (int a = 0; a < 2; ++a) {
#pragma unroll
            for (int r = 0; r < 4; ++r) d1[a][r] = h1[a][r] > 0.f ? d1[a][r] : 0.f;
            gb1 += d1[a];
            *(f4 *)&sd1[16 * a + col][u0] = d1[a];
        }
#pragma unroll
        for (int k = 0; k < kTile / 4; ++k) {
            const uint32_t s = kTile / 4 * g + k;
            const float da = sd2[s][16 * w + col];
#pragma unroll
            for (int t = 0; t < 4; ++t) gw2[t] = mfma4(da, sh1[s][16 * t + col], gw2[t]);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kTile / 4; ++k) {
            const uint32_t s = kTile / 4 * g + k;
            gw1 = mfma4(sd1[s][16 * w + col], sx[s][col], gw1);
        }
        __syncthreads();  // before the next tile's rows
    }
    float *pg = partial + (size_t)blockIdx.x * kParams;
    // sums over the 16 sample columns
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            gb1[r] += __shfl_xor(gb1[r], off, 64);
            gb2[r] += __shfl_xor(gb2[r], off, 64);
            gw3[r] += __shfl_xor(gw3[r], off, 64);
        }
        gb3 += __shfl_xor(gb3, off, 64);
        loss += __shfl_xor(loss, off, 64);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        pg[oW1 + (u0 + r) * kIn + col] = gw1[r];
#pragma unroll
        for (int t = 0; t < 4; ++t) pg[oW2 + (u0 + r) * kH + 16 * t + col] = gw2[t][r];
        if (col == 0) {
            pg[oB1 + u0 + r] = gb1[r];
            pg[oB2 + u0 + r] = gb2[r];
            pg[oW3 + u0 + r] = gw3[r];
        }
    }
    if (threadIdx.x == 0) {
        pg[oB3] = gb3;
        loss_partial[blockIdx.x] = loss;
    }
}

// Sums the partial gradients in a fixed order and applies one Adam step: 64
// parameters per workgroup, 16 threads each taking every 16th partial, their
// sums added in order through LDS (3.5 us for 128 partials; one thread
// per parameter, its loads in sequence, took 18 us for 64).
constexpr int kAdamParts = 16;
__global__ void __launch_bounds__(64 * kAdamParts)
k_mlp_adam(const float *__restrict__ partial, int nblk, float *__restrict__ params,
           float *__restrict__ m, float *__restrict__ v, float lr, float c1, float c2,
           const float *__restrict__ loss_partial, float *__restrict__ loss,
           float *__restrict__ grad) {
    __shared__ float sg[kAdamParts][64];
    const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + lane;
    float s = 0.f;
    if (p < kParams) {
#pragma unroll 8
        for (int b = part; b < nblk; b += kAdamParts) s += partial[(size_t)b * kParams + p];
    }
    sg[part][lane] = s;
    if (blockIdx.x == 0 && part == kAdamParts - 1 && loss) {
        float l = 0.f;
        for (int b = lane; b < nblk; b += 64) l += loss_partial[b];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
        if (lane == 0) loss[0] = l;
    }
    __syncthreads();
    if (part != 0 || p >= kParams) return;
    float g = 0.f;
#pragma unroll
    for (int q = 0; q < kAdamParts; ++q) g += sg[q][lane];
    if (grad) grad[p] = g;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float mn = b1 * m[p] + (1.f - b1) * g;
    const float vn = b2 * v[p] + (1.f - b2) * g * g;
    m[p] = mn;
    v[p] = vn;
    params[p] -= lr * (mn * c1) / (sqrtf(vn * c2) + eps);
}

// x[u * 16 + j] = ln(lifted[j * n + u] / n): one node per thread, so that
// every array of sizes is read in order, and a node's 16 features written as
// four 16-byte units where x starts on 16 bytes (10^6 nodes: 25 us,
// 5.0 TB/s; 41 us with one feature per thread, whose reads jump n apart).
__global__ void __launch_bounds__(256)
k_mlp_features(uint32_t n, const int32_t *__restrict__ lifted, float *__restrict__ x) {
    const float inv = 1.f / (float)n;
    const bool wide = on16(x);
    for (uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n;
         u += (uint64_t)gridDim.x * blockDim.x) {
        int32_t s[kIn];
#pragma unroll
        for (int j = 0; j < kIn; ++j) s[j] = lifted[(size_t)j * n + u];
        float *row = x + (size_t)u * kIn;
#pragma unroll
        for (int j = 0; j < kIn; j += 4) {
            f4 v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = logf((float)s[j + r] * inv);
            if (wide) {
                *(f4 *)(row + j) = v;
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) row[j + r] = v[r];
            }
        }
    }
}

// Seeded initial parameters: He-uniform weights, zero biases.  Weight p of
// the packed vector takes the p-th output of a SplitMix64 generator seeded
// with `seed` (Steele, Lea and Flood, 2014): state seed + (p + 1) * gamma,
// then the generator's output mix.  Each index is computed on its own, so
// the result does not depend on the launch shape.  The top 24 bits give
// u in [0, 1); the weight is (2u - 1) * bound in fp64, rounded to float once.
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t p) {
    uint64_t z = seed + (p + 1) * 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

__global__ void __launch_bounds__(256)
k_mlp_init(uint64_t seed, double bound1, double bound2, double bound3, float *__restrict__ params) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= kParams) return;
    double bound;
    if (p < oB1) bound = bound1;
    else if (p >= oW2 && p < oB2) bound = bound2;
    else if (p >= oW3 && p < oB3) bound = bound3;
    else {
        params[p] = 0.f;  // a bias
        return;
    }
    const double u = (double)(splitmix64_at(seed, (uint64_t)p) >> 40) * 0x1p-24;
    params[p] = (float)((2.0 * u - 1.0) * bound);
}

}  // namespace

int mlp_param_count() { return kParams; }

namespace {
// Wavefronts stay for as many tiles as it takes: at most two per SIMD of 256
// CUs, what their registers (176) leave room for, so that all run at once.
// 10^6 samples: 110 us with 512 workgroups, 140 with 768; held to 168
// registers 113 us with 768, to 128 (it spills) 173 us with 1024.
uint32_t output_blocks(int64_t N) { return (uint32_t)std::min<int64_t>((N + 63) / 64, 512); }
}  // namespace

hipError_t launch_mlp_forward(const float *params, const float *x, int64_t N, float *yhat,
                              hipStream_t st) {
    if (N <= 0) return hipSuccess;
    auto k = ((uintptr_t)x & 15u) == 0 ? k_mlp_outputs<false, true, false>
                                       : k_mlp_outputs<false, false, false>;
    hipLaunchKernelGGL(k, dim3(output_blocks(N)), dim3(256), 0, st, params, x, N,
                       0u, (const int32_t *)nullptr, yhat);
    return hipGetLastError();
}

hipError_t launch_mlp_predict(const float *params, const float *x, int64_t N, uint32_t n_nodes,
                              const int32_t *est, float *sizes, hipStream_t st) {
    if (N <= 0) return hipSuccess;
    const bool wide = ((uintptr_t)x & 15u) == 0;
    auto k = wide ? (est ? k_mlp_outputs<true, true, true> : k_mlp_outputs<true, true, false>)
                  : (est ? k_mlp_outputs<true, false, true> : k_mlp_outputs<true, false, false>);
    hipLaunchKernelGGL(k, dim3(output_blocks(N)), dim3(256), 0, st, params, x, N,
                       n_nodes, est, sizes);
    return hipGetLastError();
}

int mlp_backward_blocks(int64_t N) {
    return (int)std::min<int64_t>((N + kTile - 1) / kTile, kMaxPartials);
}

hipError_t launch_mlp_backward(const float *params, const float *x, const float *y,
                               const int32_t *idx, int64_t N, float *partial, float *loss_partial,
                               hipStream_t st) {
    hipLaunchKernelGGL(k_mlp_backward, dim3((uint32_t)mlp_backward_blocks(N)), dim3(256), 0, st,
                       params, x, y, idx, N, partial, loss_partial);
    return hipGetLastError();
}

hipError_t launch_mlp_adam(const float *partial, int nblk, float *params, float *m, float *v,
                           float lr, float c1, float c2, const float *loss_partial, float *loss,
                           float *grad, hipStream_t st) {
    hipLaunchKernelGGL(k_mlp_adam, dim3((kParams + 63) / 64), dim3(64 * kAdamParts), 0, st, partial,
                       nblk, params, m, v, lr, c1, c2, loss_partial, loss, grad);
    return hipGetLastError();
}

hipError_t launch_mlp_init(uint64_t seed, float *params, hipStream_t st) {
    // sqrt(6 / fan_in) of each layer, rounded once on the host
    hipLaunchKernelGGL(k_mlp_init, dim3((kParams + 255) / 256), dim3(256), 0, st, seed,
                       std::sqrt(6.0 / kIn), std::sqrt(6.0 / kH), std::sqrt(6.0 / kH), params);
    return hipGetLastError();
}

hipError_t launch_mlp_features(uint32_t n, uint32_t H, const int32_t *lifted, float *x,
                               hipStream_t st) {
    if (H != kIn) return hipErrorInvalidValue;
    const size_t g = std::min<size_t>(((size_t)n + 255) / 256, 65536);
    hipLaunchKernelGGL(k_mlp_features, dim3((uint32_t)g), dim3(256), 0, st, n, lifted, x);
    return hipGetLastError();
}

}  // namespace tn

// ---- training step without allocation --------------------------------------
//
// The partial gradients and losses of one training step live in a file-scope
// device array instead of the context's scratch, so that callers that cannot
// allocate (code under HIP graph capture, serving loops) can train.  Each GPU
// holds its own copy until the process ends.  In host code the array's name
// is only a stand-in for the symbol: its device address is looked up once
// per device (hipGetSymbolAddress, from tn_create) and only that address is
// passed to kernels.  Every partial the Adam kernel reads is written first by
// the backward kernel of the same call, so nothing needs clearing; calls that
// overlap on one GPU share the array and race.
namespace {
constexpr int64_t kNoAllocMaxSamples = 16384;
constexpr int kNoAllocBlocks = tn::kMaxPartials;  // partials of a step at most
static __device__ __align__(256) float scratch[(size_t)kNoAllocBlocks * (5313 + 1)];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

namespace tn {
// Looks up the array's address on the current device (once per device).
hipError_t mlp_noalloc_bind(int device) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_ptr[device]) return hipSuccess;
    float *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = ptr;
    return hipSuccess;
}
}  // namespace tn

extern "C" tn_status tn_mlp_train_step_noalloc(tn_ctx *ctx, float *params, float *adam_m,
                                               float *adam_v, int64_t step, const float *x,
                                               const float *y, const int32_t *idx, int64_t N,
                                               float lr, float *loss, float *grad) {
    using namespace tn;
    if (!ctx || !params || !adam_m || !adam_v || !x || !y) return fail(TN_E_ARG, "null argument");
    if (N <= 0) return fail(TN_E_ARG, "N must be > 0");
    if (N > kNoAllocMaxSamples)
        return fail(TN_E_UNSUPPORTED, "tn_mlp_train_step_noalloc takes at most 16384 samples per step");
    if (step < 1) return fail(TN_E_ARG, "step is 1-based");
    if (!(lr > 0.f)) return fail(TN_E_ARG, "lr must be > 0");
    if (ctx->device < 0 || ctx->device >= kMaxDevices) return fail(TN_E_ARG, "device out of range");
    float *partial;
    {
        std::lock_guard<std::mutex> lk(g_scratch_mu);
        partial = g_scratch_ptr[ctx->device];
    }
    if (!partial) return fail(TN_E_HIP, "the static training scratch of this device is not bound");
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(TN_E_HIP, "cannot select the context's device");
    const int nblk = mlp_backward_blocks(N);
    static_assert(kParams == 5313, "array size");
    float *loss_partial = partial + (size_t)nblk * kParams;
    const float c1 = (float)(1.0 / (1.0 - std::pow(0.9, (double)step)));
    const float c2 = (float)(1.0 / (1.0 - std::pow(0.999, (double)step)));
    hipError_t e;
    {
        ProfScope ps(ctx, TN_K_MLP_BACKWARD);
        e = launch_mlp_backward(params, x, y, idx, N, partial, loss_partial, ctx->stream);
    }
    if (e != hipSuccess) return hip_fail(e, "backward kernel launch");
    {
        ProfScope ps(ctx, TN_K_MLP_ADAM);
        e = launch_mlp_adam(partial, nblk, params, adam_m, adam_v, lr, c1, c2, loss_partial, loss,
                            grad, ctx->stream);
    }
    return e == hipSuccess ? TN_OK : hip_fail(e, "Adam kernel launch");
}

