// Psi1 = exp(lp1 - 1/2 sum_q w1 (mu - z)^2) on the vector unit, as a device function
// that other kernels run in workgroups of their own beside their work (one launch
// less per call).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gpps {

// 64 x 64 blocks of (n, m), a thread 4 x 4 of them, 16 dimensions staged in LDS at a
// time: twelve LDS reads serve the 48 operations of a dimension.  One thread per
// entry, reading its rows from memory, waited for each of its loads: 967 us at
// N = 100,000, M = 256, Q = 20 in fp64, against 113 us here (0.4 GB moved).
constexpr int kPsi1Tile = 64, kPsi1Q = 16;

template <typename T>
struct Psi1Lds {
    T x[kPsi1Tile][kPsi1Q + 1], w[kPsi1Tile][kPsi1Q + 1], z[kPsi1Tile][kPsi1Q + 1];
};

// Workgroups of 256 threads: block `b` of `blocks`.
template <typename T, typename Exp>
__device__ inline void psi1_blocks(Psi1Lds<T> &s, int64_t b, int64_t blocks, int64_t N, int M, int Q,
                                   const T *__restrict__ mu, const T *__restrict__ Z,
                                   const T *__restrict__ w1, const T *__restrict__ lp1,
                                   T *__restrict__ Psi1, Exp expf_) {
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int64_t mt = (M + kPsi1Tile - 1) / kPsi1Tile, nt = (N + kPsi1Tile - 1) / kPsi1Tile;
    for (int64_t t = b; t < mt * nt; t += blocks) {
        const int m0 = (int)(t % mt) * kPsi1Tile;
        const int64_t n0 = t / mt * kPsi1Tile;
        T e[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) e[i][j] = 0;
        for (int q0 = 0; q0 < Q; q0 += kPsi1Q) {
            const int qn = min(kPsi1Q, Q - q0);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kPsi1Tile * kPsi1Q / 256; ++u) {
                const int i = tid + u * 256, r = i / kPsi1Q, q = min(i % kPsi1Q, qn - 1);
                const int64_t n = min<int64_t>(n0 + r, N - 1);
                s.x[r][i % kPsi1Q] = mu[n * Q + q0 + q];
                s.w[r][i % kPsi1Q] = w1[n * Q + q0 + q];
                s.z[r][i % kPsi1Q] = Z[(int64_t)min(m0 + r, M - 1) * Q + q0 + q];
            }
            __syncthreads();
            for (int q = 0; q < qn; ++q) {
                T z[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) z[j] = s.z[tx + 16 * j][q];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const T x = s.x[4 * ty + i][q], w = s.w[4 * ty + i][q];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const T d = x - z[j];
                        e[i][j] += d * d * w;
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t n = n0 + 4 * ty + i;
            if (n >= N) break;
            const T l = lp1[n];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int m = m0 + tx + 16 * j;
                if (m < M) Psi1[n * M + m] = expf_(l - T(0.5) * e[i][j]);
            }
        }
    }
}

// Workgroups for an N x M Psi1 (0 without one), at most `cap`.
inline int64_t psi1_grid(int64_t N, int64_t M, const void *Psi1, int64_t cap) {
    if (!Psi1) return 0;
    const int64_t t = ((M + kPsi1Tile - 1) / kPsi1Tile) * ((N + kPsi1Tile - 1) / kPsi1Tile);
    return t < cap ? t : cap;
}

}  // namespace gpps
