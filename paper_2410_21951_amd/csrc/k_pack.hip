#include <algorithm>

#include "common.h"

// ---------------------------------------------------------------------------
// weight preparation: fp32 [N][K] row-major -> packed bf16 tiles
// [n-tile][k-step][lane][8]; lane (c, g) of tile (nt, ks) holds
// W[nt*16 + c][ks*32 + 8g .. 8g+7] (times gamma[k] for LN-folded maps).
// Rows >= N are zero.
// ---------------------------------------------------------------------------
__global__ void k_pack_w(const float* __restrict__ src, const float* __restrict__ gamma, uint4* __restrict__ dst,
                         int N, int K) {
    const int nks = K >> 5;
    const size_t total = (size_t)((N + 15) / 16) * nks * 64;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
        const int lane = (int)(i & 63);
        const size_t tile = i >> 6;
        const int ks = (int)(tile % nks), nt = (int)(tile / nks);
        const int n = nt * 16 + (lane & 15), k0 = ks * 32 + 8 * (lane >> 4);
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float lo = 0.f, hi = 0.f;
            if (n < N) {
                lo = src[(size_t)n * K + k0 + 2 * j];
                hi = src[(size_t)n * K + k0 + 2 * j + 1];
                if (gamma) { lo *= gamma[k0 + 2 * j]; hi *= gamma[k0 + 2 * j + 1]; }
            }
            w[j] = (uint32_t)f2bf(lo) | ((uint32_t)f2bf(hi) << 16);
        }
        dst[i] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// colsum[n] = sum_k bf16(gamma[k] W[n][k]),  tvec[n] = sum_k beta[k] W[n][k]; one wave per n
__global__ void k_fold_vectors(const float* __restrict__ src, const float* __restrict__ gamma,
                               const float* __restrict__ beta, float* __restrict__ colsum, float* __restrict__ tvec,
                               int N, int K) {
    const int n = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (n >= N) return;
    float cs = 0.f, tv = 0.f;
    for (int k = lane; k < K; k += 64) {
        const float w = src[(size_t)n * K + k];
        cs += bf2f(f2bf(w * gamma[k]));
        tv += beta[k] * w;
    }
    cs = wave_sum(cs);
    tv = wave_sum(tv);
    if (lane == 0) { colsum[n] = cs; tvec[n] = tv; }
}

__global__ void k_add_vec(float* __restrict__ dst, const float* __restrict__ src, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] += src[i];
}

void launch_pack_w(const float* src, void* dst, int N, int K, hipStream_t st) {
    const size_t total = (size_t)((N + 15) / 16) * (K >> 5) * 64;
    const int blocks = (int)std::min<size_t>((total + 255) / 256, 4096);
    launch(k_pack_w, dim3(blocks), dim3(256), 0, st, src, (const float*)nullptr, (uint4*)dst, N, K);
}

void launch_pack_w_ln(const float* src, const float* gamma, const float* beta, void* dst, float* colsum,
                      float* tvec, int N, int K, hipStream_t st) {
    const size_t total = (size_t)((N + 15) / 16) * (K >> 5) * 64;
    const int blocks = (int)std::min<size_t>((total + 255) / 256, 4096);
    launch(k_pack_w, dim3(blocks), dim3(256), 0, st, src, gamma, (uint4*)dst, N, K);
    launch(k_fold_vectors, dim3((N + 3) / 4), dim3(256), 0, st, src, gamma, beta, colsum, tvec, N, K);
}

void launch_add_vec(float* dst, const float* src, int n, hipStream_t st) {
    launch(k_add_vec, dim3((n + 255) / 256), dim3(256), 0, st, dst, src, n);
}
