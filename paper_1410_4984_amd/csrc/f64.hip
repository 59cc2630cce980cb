// Double-precision Psi2 and its gradients on the matrix cores
// (v_mfma_f64_16x16x4f64 and v_mfma_f64_4x4x4f64).
//
// With d_m = mu_n - z_m, w2 = 1 / (l^2 + 2 S_n) and lambda = log2 e, the part of
// log2 Psi2_n[m, m'] that depends on n is
//   E'_n[m, m'] = b_m + b_m' + sum_q x_mq d_m'q,
//   x_mq = -lambda/2 w2 d_mq,   b_m = lambda/2 lp2_n + 1/2 sum_q x_mq d_mq,
// and the rest, -lambda sum_q (z_m - z_m')^2 / (4 l^2), is a factor per pair:
// Psi2 = 2^C o sum_n 2^E'_n, and in the gradient it is folded into dL/dPsi2
// (Gc = G2s o 2^C).  Both operands of the contraction are local differences, so
// no term is larger than the exponents of the pairs that matter: where
// d_m ~ -d_m' makes b_m cancel against the product, C is more negative than
// either.
//
// What bounds these kernels is the vector unit's double-precision issue rate.
// A 16 x 16 x 4 product occupies a SIMD for 64 cycles and no vector
// instruction issues meanwhile (measured: 8 FMAs behind each product add 8 FMAs'
// time), so matrix and vector work add up: a matrix FMA costs the same as a
// vector one, but needs one operand load per 16 of them, no cross-lane sums and
// no index arithmetic.  The exponential is 2^E' in 15 instructions (the table's
// ln 2 is folded into x and b), against about 21 of exp().
//
// Measured against the vector kernels (fp64, psi2 gradient + forward): 45.3 + 10.6 ms
// -> 14.8 + 5.0 ms at N = 100,000, M = 256, Q = 20; 3.34 + 0.53 -> 1.43 + 0.48 ms at
// N = 50,000, M = 100, Q = 10; 261 + 3.7 -> 3.3 + 1.2 ms at N = 4096, M = 512, Q = 30.
// At the first shape the SIMDs' issue is 40% matrix and 30-40% vector instructions.
//
// Rows whose exponents leave the range in which that is exact (|b| < 2^26: means
// thousands of lengthscales from an inducing input, infinities, NaN) take a
// direct evaluation of each pair, on a branch that is uniform over a wave.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "psi1.h"

namespace gpps {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr size_t kLdsMax = 160 * 1024;
constexpr int kSimds = 1024;   // 256 CUs x 4
constexpr double kLog2e = 1.4426950408889634074;
constexpr double kSlow = 67108864.0;  // 2^26: the largest |b| of the fast exponential

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

__device__ inline d4 mfma16(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// Sum over the four lane groups (lanes l, l + 16, l + 32, l + 48), in every lane.
__device__ inline double sum_groups(double v) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, v, 0.0, 0, 0, 0);
}

// 2^x for |x| < 2^31: x = n + f with n the nearest integer, 2^f by a polynomial of
// degree 11 with constant term 1 (minimax in the relative error over |f| <= 1/2,
// 4.2e-17 after rounding its coefficients; 1.4e-16 with the rounding of Horner's
// rule), scaled by ldexp, which underflows to zero.
__device__ inline double exp2_fast(double x) {
    const double magic = 0x1.8p52;
    const double t = x + magic;
    const int n = (int)(unsigned)__double_as_longlong(t);
    const double f = x - (t - magic);
    double p = 0x1.c0638527edf3ep-32;
    p = fma(p, f, 0x1.e605f979c7a84p-28);
    p = fma(p, f, 0x1.b54167a0b9065p-24);
    p = fma(p, f, 0x1.62bfd49ed0adfp-20);
    p = fma(p, f, 0x1.ffcbee3b0af8cp-17);
    p = fma(p, f, 0x1.4309130961163p-13);
    p = fma(p, f, 0x1.5d87fe7bbbe07p-10);
    p = fma(p, f, 0x1.3b2ab6fba1e1cp-7);
    p = fma(p, f, 0x1.c6b08d7048f31p-5);
    p = fma(p, f, 0x1.ebfbdff82c598p-3);
    p = fma(p, f, 0x1.62e42fefa39f3p-1);
    p = fma(p, f, 1.0);
    return __builtin_amdgcn_ldexp(p, n);
}

// Psi2_n[m, m'] without the pair factor, by the closed form itself (slow rows).
__device__ inline double direct_pair(const double *__restrict__ x, const double *__restrict__ w2,
                                     double lp2, const double *__restrict__ za,
                                     const double *__restrict__ zb, int Q) {
    double e = lp2;
    for (int q = 0; q < Q; ++q) {
        const double d = x[q] - 0.5 * (za[q] + zb[q]);
        e -= d * d * w2[q];
    }
    return exp(e);
}

// LDS written by lanes of this wave is read by others of it: a wave's LDS operations
// complete in order, so only the compiler has to keep theirs.
__device__ inline void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------- forward
// A wave owns C blocks of 16 columns m and up to A blocks of 16 rows m' at or past
// them (4 and 2 up to Q = 32), and sums its tiles over the rows n of a chunk.  Its
// z rows stay in registers as differences' constants; per row n it forms d for
// its blocks, x for its columns and b for all, which is shared by its
// tiles.  b of a row block is summed over q by one product with ones,
// which leaves it in the tile's own layout.
constexpr int kFwdMinRows = 4;   // rows per chunk of the smallest calls (a row takes a wave 2 us alone)
constexpr int kFwdFlush = 128;  // rows summed before they join the chunk's total

// Row and column blocks of a task: as many as leave its z rows, x and sums within
// 256 registers.
__host__ __device__ constexpr int fwd_a(int ks) { return ks <= 8 ? 4 : 2; }
__host__ __device__ constexpr int fwd_c(int ks) { return ks <= 12 ? 2 : 1; }
// Rows n staged at a time, per wave in two buffers (eight waves share a CU's LDS).
__host__ __device__ constexpr int fwd_rows(int ks) { return ks <= 8 ? 16 : 8; }

constexpr int kFwdWaves = 4;   // waves per workgroup (one per SIMD; they share nothing)

// The tasks of the upper triangle of nb blocks: for each column group the groups of
// A row blocks at or below it.  A task gets row chunks in proportion to its tiles
// (and the work per row that its tiles share, about a tile's), cmax for one with
// all A C tiles, so that every wave takes the same time and one round of two
// waves per SIMD has no tail; the waves are numbered task by task.
struct FwdTask {
    int cb, rb;        // first column and row block
    int first, chunks; // its waves
};
__host__ __device__ inline int fwd_tiles(int nb, int A, int C, int cb, int rb) {
    const int na = nb - rb < A ? nb - rb : A, nc = nb - cb < C ? nb - cb : C;
    int tiles = 0;
    for (int a = 0; a < na; ++a) {
        const int up = rb + a - cb + 1;  // column blocks at or above the diagonal
        tiles += up < nc ? up : nc;
    }
    return tiles;
}
__host__ __device__ inline int fwd_chunks(int64_t N, int nb, int A, int C, int cb, int rb, int cmax) {
    const int n = cmax * (fwd_tiles(nb, A, C, cb, rb) + 1) / (A * C + 1);
    return n < 1 ? 1 : n > N ? (int)N : n;
}
// The task that holds wave w, or the one numbered `task` (the other is negative).
__device__ inline FwdTask fwd_task(int64_t N, int nb, int A, int C, int cmax, int w, int task) {
    FwdTask t{0, 0, 0, 0};
    for (t.cb = 0; t.cb < nb; t.cb += C)
        for (t.rb = t.cb; t.rb < nb; t.rb += A) {
            t.chunks = fwd_chunks(N, nb, A, C, t.cb, t.rb, cmax);
            if (w >= 0 ? w < t.first + t.chunks : task-- == 0) return t;
            t.first += t.chunks;
        }
    t.chunks = 0;
    return t;
}

template <int KS>
__global__ __launch_bounds__(kFwdWaves * 64, 2) void psi2_fwd_kernel(
    int64_t N, int M, int Q, int nb, int cmax, const double *__restrict__ mu,
    const double *__restrict__ Z, const double *__restrict__ w2, const double *__restrict__ lp2,
    double *__restrict__ partial) {
    constexpr int QP = 4 * KS, kFwdA = fwd_a(KS), kFwdC = fwd_c(KS), kFwdRows = fwd_rows(KS);
    __shared__ double t_mu[kFwdWaves][2][kFwdRows][QP], t_k[kFwdWaves][2][kFwdRows][QP],
        t_h[kFwdWaves][2][kFwdRows];
    const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto &s_mu = t_mu[wv];
    auto &s_k = t_k[wv];
    auto &s_h = t_h[wv];
    const int w = blockIdx.x * kFwdWaves + wv;
    const FwdTask task = fwd_task(N, nb, kFwdA, kFwdC, cmax, w, -1);
    if (task.chunks == 0) return;
    const int cb = task.cb, rb = task.rb, na = min(kFwdA, nb - rb);
    // blocks past the edge repeat the last inducing input (never stored)
    double za[kFwdA][KS], zc[kFwdC][KS];
#pragma unroll
    for (int a = 0; a < kFwdA; ++a) {
        const int m = min((rb + a) * 16 + c16, M - 1);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int q = 4 * s + g;
            const double v = Z[(int64_t)m * Q + min(q, Q - 1)];
            za[a][s] = q < Q ? v : 0.0;
        }
    }
#pragma unroll
    for (int c = 0; c < kFwdC; ++c) {
        const int m = min((cb + c) * 16 + c16, M - 1);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int q = 4 * s + g;
            const double v = Z[(int64_t)m * Q + min(q, Q - 1)];
            zc[c][s] = q < Q ? v : 0.0;
        }
    }
    d4 acc[kFwdA][kFwdC];
#pragma unroll
    for (int a = 0; a < kFwdA; ++a)
#pragma unroll
        for (int c = 0; c < kFwdC; ++c) acc[a][c] = d4{0, 0, 0, 0};
    const int64_t r0 = N * (w - task.first) / task.chunks, r1 = N * (w - task.first + 1) / task.chunks;
    // partial[wave][tile][v][lane]
    double *out = partial + (int64_t)w * (kFwdA * kFwdC * 256) + lane;
    auto stage = [&](int64_t base, int buf) {
        const int cnt = (int)min<int64_t>(kFwdRows, r1 - base);
        for (int i = lane; i < kFwdRows * QP; i += 64) {
            const int r = i / QP, q = i - r * QP;
            const int64_t n = base + min(r, cnt - 1);
            const double m = mu[n * Q + min(q, Q - 1)], w = w2[n * Q + min(q, Q - 1)];
            s_mu[buf][r][q] = q < Q ? m : 0.0;
            s_k[buf][r][q] = q < Q ? -0.5 * kLog2e * w : 0.0;
        }
        if (lane < kFwdRows) s_h[buf][lane] = 0.125 * kLog2e * lp2[base + min(lane, cnt - 1)];
    };
    int flushed = 0;
    if (r0 < r1) stage(r0, 0);
    int buf = 0;
    for (int64_t base = r0; base < r1; base += kFwdRows, buf ^= 1) {
        const int cnt = (int)min<int64_t>(kFwdRows, r1 - base);
        wave_lds_fence();
        if (base + kFwdRows < r1) stage(base + kFwdRows, buf ^ 1);
        for (int r = 0; r < cnt; ++r) {
            const double hl = s_h[buf][r];  // a quarter of lambda/2 lp2: one per lane group
            double muq[KS], kq[KS];
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                muq[s] = s_mu[buf][r][4 * s + g];
                kq[s] = s_k[buf][r][4 * s + g];
            }
            double x[kFwdC][KS], bc[kFwdC];
            bool ok = true;
#pragma unroll
            for (int c = 0; c < kFwdC; ++c) {
                double part = 0.0;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const double d = muq[s] - zc[c][s];
                    x[c][s] = kq[s] * d;
                    part = fma(x[c][s], d, part);
                }
                part = fma(0.5, part, hl);
                ok = ok && fabs(part) < 0.25 * kSlow;
                bc[c] = sum_groups(part);
            }
#pragma unroll
            for (int a = 0; a < kFwdA; ++a) {
                if (a >= na) break;  // uniform
                __builtin_amdgcn_sched_barrier(0);
                double da[KS], part = 0.0;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    da[s] = muq[s] - za[a][s];
                    part = fma(kq[s] * da[s], da[s], part);
                }
                part = fma(0.5, part, hl);
                if (__builtin_expect(__all(ok && fabs(part) < 0.25 * kSlow), 1)) {
                    const d4 br = mfma16(part, 1.0, d4{0, 0, 0, 0});
#pragma unroll
                    for (int c = 0; c < kFwdC; ++c) {
                        if (cb + c > rb + a || cb + c >= nb) break;  // uniform: below the diagonal
                        d4 e;
#pragma unroll
                        for (int v = 0; v < 4; ++v) e[v] = br[v] + bc[c];
#pragma unroll
                        for (int s = 0; s < KS; ++s) e = mfma16(da[s], x[c][s], e);
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[a][c][v] += exp2_fast(e[v]);
                    }
                } else {
                    const int64_t n = base + r;
                    int l = lane;  // opaque: nothing of this branch is kept in registers outside it
                    asm volatile("" : "+v"(l));
#pragma unroll
                    for (int c = 0; c < kFwdC; ++c)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int m = min((cb + c) * 16 + (l & 15), M - 1);
                            const int mp = min((rb + a) * 16 + 4 * v + (l >> 4), M - 1);
                            __builtin_amdgcn_sched_barrier(0);
                            acc[a][c][v] += direct_pair(mu + n * Q, w2 + n * Q, lp2[n],
                                                        Z + (int64_t)m * Q, Z + (int64_t)mp * Q, Q);
                        }
                }
            }
        }
        // two-level sum: 128 rows, then into the chunk's total in HBM, so that
        // rounding does not grow with the rows of a chunk
        const bool last = base + kFwdRows >= r1;
        if (last || (base + kFwdRows - r0) % kFwdFlush == 0) {
#pragma unroll
            for (int a = 0; a < kFwdA; ++a)
#pragma unroll
                for (int c = 0; c < kFwdC; ++c)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        double *o = out + ((a * kFwdC + c) * 4 + v) * 64;
                        *o = flushed ? *o + acc[a][c][v] : acc[a][c][v];
                        acc[a][c][v] = 0.0;
                    }
            flushed = 1;
        }
    }
}

// Workgroups below tasks A C: Psi2[m, m'] = 2^C sum over chunks, in chunk order, one
// tile of a task each, one thread per entry; both triangles and psi0.  The
// workgroups past them compute Psi1.
__global__ __launch_bounds__(256) void psi2_fwd_reduce_kernel(
    int64_t N, int M, int Q, int nb, int A, int CB, int cmax, int tasks,
    const double *__restrict__ partial, const double *__restrict__ Z, Hyp<double> h,
    double *__restrict__ psi0, double *__restrict__ Psi2, int accumulate,
    const double *__restrict__ mu, const double *__restrict__ w1, const double *__restrict__ lp1,
    double *__restrict__ Psi1) {
    __shared__ Psi1Lds<double> s_p1;
    const unsigned rblocks = tasks * A * CB;
    if (blockIdx.x >= rblocks) {
        psi1_blocks<double>(s_p1, blockIdx.x - rblocks, gridDim.x - rblocks, N, M, Q, mu, Z, w1, lp1, Psi1,
                            [](double x) { return exp(x); });
        return;
    }
    const int tile = blockIdx.x % (A * CB);
    if (blockIdx.x == 0 && threadIdx.x == 0)
        psi0[0] = (accumulate ? psi0[0] : 0.0) + (double)N * h.sf2;
    const FwdTask task = fwd_task(N, nb, A, CB, cmax, -1, blockIdx.x / (A * CB));
    const int cb = task.cb + tile % CB, rb = task.rb + tile / CB, chunks = task.chunks;
    if (cb >= nb || rb >= nb || cb > rb) return;
    const int lane = threadIdx.x & 63, v = threadIdx.x >> 6;
    const int m = cb * 16 + (lane & 15), mp = rb * 16 + 4 * v + (lane >> 4);
    if (m >= M || mp >= M || m > mp) return;
    const int64_t stride = A * CB * 256;
    const double *src = partial + task.first * stride + tile * 256 + threadIdx.x;
    double s = 0.0;
    int k = 0;
    for (; k + 8 <= chunks; k += 8) {
        double t[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = src[(k + j) * stride];
#pragma unroll
        for (int j = 0; j < 8; ++j) s += t[j];
    }
    for (; k < chunks; ++k) s += src[k * stride];
    double C = 0.0;
    for (int q = 0; q < Q; ++q) {
        const double dz = Z[(int64_t)m * Q + q] - Z[(int64_t)mp * Q + q];
        C -= dz * dz / (4.0 * h.l2[q]);
    }
    const double val = (accumulate ? Psi2[(int64_t)m * M + mp] : 0.0) + exp(C) * s;
    Psi2[(int64_t)m * M + mp] = val;
    Psi2[(int64_t)mp * M + m] = val;
}

// ---------------------------------------------------------------- gradient
template <int CTRL>
__device__ inline double rotate16(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// Sums within the 16 lanes of a lane group: over the lanes of equal lane & 3, and
// over all of them; in every lane.
__device__ inline double sum_fours(double v) {
    v += rotate16<0x128>(v);  // row_ror:8
    v += rotate16<0x124>(v);
    return v;
}
__device__ inline double sum16(double v) {
    v = sum_fours(v);
    v += rotate16<0x122>(v);
    v += rotate16<0x121>(v);
    return v;
}

// Rows n a wave works on at once: as many as keep x, V and the row values of
// 2 R (row, column block) pairs within 256 registers.
template <int KS>
constexpr int grad_rows() { return KS <= 5 ? 2 : 1; }

struct GradGeo {
    int nw;          // waves per workgroup (each two column blocks)
    int wrows;       // z rows staged at a time (a multiple of 16)
    int nwin;        // windows of wrows rows
    int64_t chunks, rows;
    int groups;      // workgroups per row chunk
    size_t lds;
};

constexpr int kGradC = 2;      // column blocks per wave

// With W_n = Gc o 2^E'_n, r_m = sum_m' W, V_m = sum_m' W d_m', t = dL/dPsi1 o Psi1,
// every gradient is a sum over (n, m) of terms in (r, V, t) (the formulas stand at
// the generic pairs kernel).  A wave owns 32 columns m and walks the blocks of
// 16 rows m': a tile of W leaves the exponent's product in exactly the layout
// that the second product, V^T += d^T W, takes as its right operand, and V comes
// out in the layout of x, so neither goes through LDS.  Each (m', d, Gc) operand
// serves 2 R products.  r is summed on the vector unit: 4 additions a tile, where a
// column of ones would cost 64 cycles.  Sums over m (dmu, dS, dl) go through the
// lanes and then the waves in a fixed order; dZ stays in LDS slots that one lane
// owns.
template <int KS>
__global__ __launch_bounds__(512) void psi2_grad_kernel(
    int64_t N, int M, int Q, int nb, int wrows, int nwin, int64_t rows_per_chunk,
    const double *__restrict__ mu, const double *__restrict__ S, const double *__restrict__ Z,
    const double *__restrict__ w1t, const double *__restrict__ w2t, const double *__restrict__ lp1,
    const double *__restrict__ lp2, Hyp<double> h, const double *__restrict__ G1,
    const double *__restrict__ Gc, double *__restrict__ dmu, double *__restrict__ dS,
    double *__restrict__ colpart, double *__restrict__ rowpart) {
    constexpr int QP = 4 * KS, ZS = QP + 1, R = grad_rows<KS>(), T16 = KS / 4, T4 = KS % 4;
    constexpr int NT = T16 + T4;
    extern __shared__ double sm[];
    const int tid = threadIdx.x, nthr = blockDim.x, nw = nthr >> 6;
    const int lane = tid & 63, g = lane >> 4, c16 = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wcols = nw * kGradC * 16;
    double *sz = sm;                          // [wrows][ZS]
    double *sb = sz + wrows * ZS;             // [R][wrows]: b of the rows, permuted in each block
    double *sbc = sb + R * wrows;             // [R][wcols]: b of the workgroup's columns
    double *srow = sbc + R * wcols;           // [R][4][QP]: mu, w1, w2, S
    double *slp = srow + R * 4 * QP;          // [R][2]: lp1, lp2
    double *sred = slp + R * 2;               // [nw][R][3 QP + 2]
    double *sdl = sred + nw * R * (3 * QP + 2);  // [R][QP + 1]
    double *shyp = sdl + R * (QP + 1);        // [3][QP]: 1/l^2, l, 1/l^3
    double *sgz = shyp + 3 * QP;              // [wcols][QP]
    int *sslow = reinterpret_cast<int *>(sgz + wcols * QP);  // [2][R]
    const int Mp = nb * 16;
    const int cb0 = (blockIdx.x * nw + wv) * kGradC;       // the wave's first column block
    const int ncol = min(kGradC, nb - cb0);                // its column blocks (<= 0: none)
    const int m0 = blockIdx.x * wcols;                     // the workgroup's first column
    for (int q = tid; q < QP; q += nthr) {
        const double l = q < Q ? h.l[q] : 1.0, l2 = q < Q ? h.l2[q] : 1.0;
        shyp[q] = 1.0 / l2;
        shyp[QP + q] = l;
        shyp[2 * QP + q] = 1.0 / (l2 * l);
    }
    for (int i = tid; i < R * (QP + 1); i += nthr) sdl[i] = 0.0;
    for (int i = tid; i < wcols * QP; i += nthr) sgz[i] = 0.0;
    // rows of Z past M repeat the last one: finite wherever the real ones are
    auto stage_z = [&](int w0) {
        for (int i = tid; i < wrows * QP; i += nthr) {
            const int r = i / QP, q = i - r * QP;
            const double v = Z[(int64_t)min(w0 + r, M - 1) * Q + min(q, Q - 1)];
            sz[r * ZS + q] = q < Q ? v : 0.0;
        }
    };
    if (nwin == 1) stage_z(0);
    // coordinate q of inducing input m (any q where the row values are zero beyond Q)
    auto zcol = [&](int m, int q) {
        return nwin == 1 ? sz[m * ZS + q] : Z[(int64_t)m * Q + min(q, Q - 1)];
    };
    // this lane's Psi1 term: row lane >> 5 (R = 2) of its columns lane & 31
    const int64_t r0 = (int64_t)blockIdx.y * rows_per_chunk, r1 = min(N, r0 + rows_per_chunk);
    for (int64_t base = r0; base < r1; base += R) {
        const int cnt = (int)min<int64_t>(R, r1 - base);
        __syncthreads();
        for (int i = tid; i < R * 4 * QP; i += nthr) {
            const int r = i / (4 * QP), k = (i / QP) & 3, q = i % QP;
            const double *src = k == 0 ? mu : k == 1 ? w1t : k == 2 ? w2t : S;
            const double v = src[(base + min(r, cnt - 1)) * Q + min(q, Q - 1)];
            srow[i] = q < Q ? v : 0.0;
        }
        if (tid < R) {
            slp[2 * tid] = lp1[base + min(tid, cnt - 1)];
            slp[2 * tid + 1] = lp2[base + min(tid, cnt - 1)];
        }
        if (tid < 2 * R) sslow[tid] = 0;
        __syncthreads();
        // b of row r and inducing input m
        auto b_of = [&](int r, const double *z) {
            const double *xr = srow + r * 4 * QP, *w = xr + 2 * QP;
            double s = 0.0;
#pragma unroll 4
            for (int q = 0; q < QP; ++q) {
                const double d = xr[q] - z[min(q, Q - 1)];
                s = fma(w[q] * d, d, s);
            }
            return kLog2e * (0.5 * slp[2 * r + 1] - 0.25 * s);
        };
        // place of row j in sb: row 4 v + g of a block at 4 g + v, so that a lane's four
        // are contiguous
        auto b_at = [](int j) { return (j & ~15) + 4 * (j & 3) + ((j >> 2) & 3); };
        if (nwin > 1)  // else the columns are among the rows of the one window
            for (int i = tid; i < R * wcols; i += nthr) {
                const int r = i / wcols;
                const double s = b_of(r, Z + (int64_t)min(m0 + i - r * wcols, M - 1) * Q);
                sbc[i] = s;
                if (!(fabs(s) < kSlow)) sslow[r] = 1;
            }
        double x[R][kGradC][KS], rs[R][kGradC];
        d4 V16[R][kGradC][T16 > 0 ? T16 : 1];
        double V4[R][kGradC][T4 > 0 ? T4 : 1];
        double tval = 0.0;
        // the Psi1 terms t = dL/dPsi1 o Psi1 of (row, column) = this lane's
        if (G1) {
            const int r = R == 2 ? lane >> 5 : 0, cc = lane & 31;
            const int m = cb0 * 16 + cc;
            if (r < cnt && m < M && (R == 2 || lane < 32)) {
                const double *xr = srow + r * 4 * QP, *w = xr + QP;
                double s = 0.0;
#pragma unroll 4
                for (int q = 0; q < QP; ++q) {
                    const double d = xr[q] - zcol(m, q);
                    s = fma(w[q] * d, d, s);
                }
                tval = G1[(base + r) * M + m] * exp(slp[2 * r] - 0.5 * s);
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < kGradC; ++c) {
                rs[r][c] = 0.0;
                const int m = min((cb0 + c) * 16 + c16, M - 1);
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const int q = 4 * s + g;
                    const double d = srow[r * 4 * QP + q] - zcol(m, q);
                    x[r][c][s] = -0.5 * kLog2e * srow[r * 4 * QP + 2 * QP + q] * d;
                }
#pragma unroll
                for (int t = 0; t < T16; ++t) V16[r][c][t] = d4{0, 0, 0, 0};
#pragma unroll
                for (int t = 0; t < T4; ++t) V4[r][c][t] = 0.0;
            }
        if (Gc) {
            double bi[R][kGradC];
            for (int win = 0; win < nwin; ++win) {
                const int w0 = win * wrows;
                if (nwin > 1) {
                    if (win) __syncthreads();
                    stage_z(w0);
                    if (tid < R) sslow[R + tid] = 0;
                    __syncthreads();
                }
                for (int i = tid; i < R * wrows; i += nthr) {
                    const int r = i / wrows, j = i - r * wrows;
                    const double *xr = srow + r * 4 * QP, *w = xr + 2 * QP, *z = sz + j * ZS;
                    double s = 0.0;
#pragma unroll 4
                    for (int q = 0; q < QP; ++q) {
                        const double d = xr[q] - z[q];
                        s = fma(w[q] * d, d, s);
                    }
                    s = kLog2e * (0.5 * slp[2 * r + 1] - 0.25 * s);
                    sb[r * wrows + b_at(j)] = s;
                    if (!(fabs(s) < kSlow)) sslow[R + r] = 1;
                }
                __syncthreads();
                if (win == 0) {
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int c = 0; c < kGradC; ++c)
                            bi[r][c] = nwin == 1 ? sb[r * wrows + b_at(min((cb0 + c) * 16 + c16, Mp - 1))]
                                                 : sbc[r * wcols + (wv * kGradC + c) * 16 + c16];
                }
                if (ncol <= 0) continue;
                bool slow[R];
#pragma unroll
                for (int r = 0; r < R; ++r)
                    slow[r] = __builtin_amdgcn_readfirstlane(sslow[r] | sslow[R + r]) != 0;
                double muA[R][KS], muB[R][NT];
#pragma unroll
                for (int r = 0; r < R; ++r) {
#pragma unroll
                    for (int s = 0; s < KS; ++s) muA[r][s] = srow[r * 4 * QP + 4 * s + g];
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        muB[r][t] = srow[r * 4 * QP + (t < T16 ? 16 * t + c16
                                                               : 16 * T16 + 4 * (t - T16) + (lane & 3))];
                }
                const int jn = min(wrows, Mp - w0) / 16;
                // NC: the wave's column blocks, so that their tiles interleave
                auto tiles = [&](auto ncc) {
                    constexpr int NC = decltype(ncc)::value;
                    for (int J = 0; J < jn; ++J) {
                        double G[NC][4];
#pragma unroll
                        for (int c = 0; c < NC; ++c)
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                G[c][v] = Gc[(int64_t)(w0 + 16 * J + 4 * v + g) * Mp + (cb0 + c) * 16 + c16];
                        double zA[KS];
#pragma unroll
                        for (int s = 0; s < KS; ++s) zA[s] = sz[(16 * J + c16) * ZS + 4 * s + g];
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            __builtin_amdgcn_sched_barrier(0);
                            double W[NC][4];
                            if (__builtin_expect(!slow[r], 1)) {
                                double dA[KS];
                                d4 e[NC];
#pragma unroll
                                for (int v = 0; v < 4; ++v) {
                                    const double b = sb[r * wrows + 16 * J + 4 * g + v];
#pragma unroll
                                    for (int c = 0; c < NC; ++c) e[c][v] = b + bi[r][c];
                                }
#pragma unroll
                                for (int s = 0; s < KS; ++s) dA[s] = muA[r][s] - zA[s];
#pragma unroll
                                for (int s = 0; s < KS; ++s)
#pragma unroll
                                    for (int c = 0; c < NC; ++c) e[c] = mfma16(dA[s], x[r][c][s], e[c]);
#pragma unroll
                                for (int c = 0; c < NC; ++c)
#pragma unroll
                                    for (int v = 0; v < 4; ++v) W[c][v] = G[c][v] * exp2_fast(e[c][v]);
                            } else {
                                int l = lane;  // opaque: nothing of this branch is kept outside it
                                asm volatile("" : "+v"(l));
#pragma unroll
                                for (int c = 0; c < NC; ++c)
#pragma unroll
                                    for (int v = 0; v < 4; ++v) {
                                        const int m = (cb0 + c) * 16 + (l & 15);
                                        const int mp = w0 + 16 * J + 4 * v + (l >> 4);
                                        __builtin_amdgcn_sched_barrier(0);
                                        W[c][v] = 0.0;
                                        if (m < M && mp < M)
                                            W[c][v] = G[c][v] *
                                                      direct_pair(srow + r * 4 * QP,
                                                                  srow + r * 4 * QP + 2 * QP,
                                                                  slp[2 * r + 1], Z + (int64_t)m * Q,
                                                                  Z + (int64_t)mp * Q, Q);
                                    }
                            }
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int c = 0; c < NC; ++c)
                                rs[r][c] += (W[c][0] + W[c][1]) + (W[c][2] + W[c][3]);
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                double dB[NT];
#pragma unroll
                                for (int t = 0; t < NT; ++t)
                                    dB[t] = muB[r][t] -
                                            sz[(16 * J + 4 * v + g) * ZS +
                                               (t < T16 ? 16 * t + c16 : 16 * T16 + 4 * (t - T16) + (lane & 3))];
#pragma unroll
                                for (int c = 0; c < NC; ++c) {
#pragma unroll
                                    for (int t = 0; t < T16; ++t)
                                        V16[r][c][t] = mfma16(W[c][v], dB[t], V16[r][c][t]);
#pragma unroll
                                    for (int t = 0; t < T4; ++t)
                                        V4[r][c][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(
                                            W[c][v], dB[T16 + t], V4[r][c][t], 0, 0, 0);
                                }
                            }
                        }
                    }
                };
                if (ncol == 1)
                    tiles(std::integral_constant<int, 1>{});
                else
                    tiles(std::integral_constant<int, kGradC>{});
            }
        }
        // epilogue: of a 16-wide tile t lane (g, c16) holds (m = 4 v + g, q = 16 t + c16),
        // of a 4-wide one (m = (lane & 12) + g, q = 16 T16 + 4 t + (lane & 3))
        if (ncol > 0) {
            int le = lane;  // opaque: the epilogue's addresses are formed here, not kept over the tiles
            asm volatile("" : "+v"(le));
            const int ge = le >> 4, ce = le & 15;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (r >= cnt) break;  // uniform
                double *red = sred + (wv * R + r) * (3 * QP + 2);
                double tc[kGradC];
                d4 r16[kGradC];
                double r4[kGradC], rt = 0.0, tt = 0.0;
#pragma unroll
                for (int c = 0; c < kGradC; ++c) {
                    if (c >= ncol) rs[r][c] = 0.0;
                    tc[c] = __shfl(tval, 32 * r + 16 * c + ce);
                    rt += rs[r][c];
                    tt += tc[c];
                    if (T16 > 0) r16[c] = mfma16(rs[r][c], 1.0, d4{0, 0, 0, 0});
                    if (T4 > 0) r4[c] = __builtin_amdgcn_mfma_f64_4x4x4f64(rs[r][c], 1.0, 0.0, 0, 0, 0);
                }
                rt = sum16(sum_groups(rt));
                tt = sum16(tt);
                if (lane == 0) {
                    red[3 * QP] = rt;
                    red[3 * QP + 1] = tt;
                }
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const bool wide = t < T16;
                    const int q = wide ? 16 * t + ce : 16 * T16 + 4 * (t - T16) + (le & 3);
                    const double *row = srow + r * 4 * QP + q;
                    const double xm = row[0], a1 = row[QP], a2 = row[2 * QP];
                    const double il2 = shyp[q], l = shyp[QP + q], il3 = shyp[2 * QP + q];
                    double sp0 = 0.0, st0 = 0.0, su = 0.0, sn = 0.0, sx = 0.0;
#pragma unroll
                    for (int c = 0; c < kGradC; ++c) {
                        if (c >= ncol) break;  // uniform
#pragma unroll
                        for (int v = 0; v < (wide ? 4 : 1); ++v) {
                            const int ml = wide ? 4 * v + ge : (le & 12) + ge;
                            const int m = min((cb0 + c) * 16 + ml, M - 1);
                            const double rm = wide ? r16[c][v] : r4[c];
                            const double tm = __shfl(tval, 32 * r + 16 * c + ml);
                            const double Vq = wide ? V16[r][c][wide ? t : 0][v] : V4[r][c][wide ? 0 : t - T16];
                            const double d = xm - zcol(m, q), dr = d * rm, td = tm * d;
                            const double p = dr + Vq, n = dr - Vq;
                            sp0 += dr;
                            st0 += td;
                            su = fma(d, p, su);
                            sn = fma(d, n, sn);
                            sx = fma(d, td, sx);
                            double *gz = sgz + ((wv * kGradC + c) * 16 + ml) * QP + q;
                            *gz += fma(a2, p, fma(il2, n, a1 * td));
                        }
                    }
                    const double u = a2 * a2 * su, y = a1 * a1 * sx;
                    double v0 = sum_groups(-2.0 * a2 * sp0 - a1 * st0);
                    double v1 = sum_groups(u + 0.5 * y);
                    double v2 = sum_groups(fma(sn, il3, l * (u + y)));
                    if (!wide) {
                        v0 = sum_fours(v0);
                        v1 = sum_fours(v1);
                        v2 = sum_fours(v2);
                    }
                    if (lane < (wide ? 16 : 4)) {
                        red[q] = v0;
                        red[QP + q] = v1;
                        red[2 * QP + q] = v2;
                    }
                }
            }
        }
        __syncthreads();
        // dmu, dS of the rows (over the workgroup's columns) and the dl, dsf2 terms
        const int live = min(nw, (nb - (int)blockIdx.x * nw * kGradC + kGradC - 1) / kGradC);
        for (int i = tid; i < cnt * Q; i += nthr) {
            const int r = i / Q, q = i - r * Q;
            double v0 = 0.0, v1 = 0.0, v2 = 0.0, Rt = 0.0, Tt = 0.0;
            for (int w = 0; w < live; ++w) {
                const double *red = sred + (w * R + r) * (3 * QP + 2);
                v0 += red[q];
                v1 += red[QP + q];
                v2 += red[2 * QP + q];
                Rt += red[3 * QP];
                Tt += red[3 * QP + 1];
            }
            const double *row = srow + r * 4 * QP + q;
            const double a1 = row[QP], a2 = row[2 * QP], sv = row[3 * QP], il = 1.0 / shyp[QP + q];
            const int64_t o = ((int64_t)blockIdx.x * 2 * N + base + r) * Q + q;
            dmu[o] = v0;
            dS[o] = v1 - a2 * Rt - 0.5 * a1 * Tt;
            sdl[r * (QP + 1) + q] += v2 + (2.0 * sv * a2 * il) * Rt + (sv * a1 * il) * Tt;
            if (q == 0) sdl[r * (QP + 1) + QP] += 2.0 * Rt + Tt;
        }
    }
    __syncthreads();
    for (int i = tid; i < wcols * Q; i += nthr) {
        const int cc = i / Q, q = i - cc * Q;
        if (m0 + cc < M) colpart[((int64_t)blockIdx.y * M + m0 + cc) * Q + q] = sgz[cc * QP + q];
    }
    for (int q = tid; q <= Q; q += nthr) {
        double s = 0.0;
        for (int r = 0; r < R; ++r) s += sdl[r * (QP + 1) + (q < Q ? q : QP)];
        rowpart[((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * (Q + 1) + q] =
            q < Q ? s : s / h.sf2;
    }
}

// k-steps of 4 dimensions, rounded to the instantiated widths
int ks_of(int64_t Q) {
    for (int ks : {1, 2, 3, 4, 5, 6, 8, 10, 12})
        if (Q <= 4 * ks) return ks;
    return 16;
}

int rows_of(int ks) { return ks <= 5 ? 2 : 1; }

size_t grad_lds(int ks, int nw, int wrows) {
    const int QP = 4 * ks, R = rows_of(ks), wcols = nw * kGradC * 16;
    const size_t d = (size_t)wrows * (QP + 1) + R * wrows + R * wcols + R * 4 * QP + R * 2 +
                     (size_t)nw * R * (3 * QP + 2) + R * (QP + 1) + 3 * QP + (size_t)wcols * QP;
    return d * 8 + 2 * R * 4 + 8;
}


GradGeo grad_geo(const Shape &s) {
    GradGeo g{};
    const int ks = ks_of(s.Q), R = rows_of(ks);
    const int nb = (int)cdiv(s.M, 16), need = (int)cdiv(nb, kGradC);  // waves per row chunk
    // the waves per workgroup that keep the most of a CU's eight wave slots (two per
    // SIMD: the register limit) on column blocks that exist, in at most one group of
    // columns per 128 (each writes dmu and dS of its own); the widest of equal ones
    double best = 0.0;
    for (int nw = std::min(8, need); nw >= 1; --nw) {
        const int groups = (int)cdiv(need, nw);
        if (groups > cdiv(nb, 8)) break;
        // Z whole in LDS where it fits, else the fewest equal windows that do
        int nwin = 1, wrows;
        size_t lds;
        for (;; ++nwin) {
            wrows = (int)cdiv(nb, nwin) * 16;
            lds = grad_lds(ks, nw, wrows);
            if (lds <= kLdsMax || wrows == 16) break;
        }
        if (lds > kLdsMax) continue;
        const int per_cu = (int)std::min<int64_t>((int64_t)(kLdsMax / lds), 8 / nw);
        const double score = (double)nb / (kGradC * nw * groups) * (per_cu * nw) / (nwin > 1 ? 1.05 : 1.0);
        if (score > 1.02 * best) {
            best = score;
            g.nw = nw;
            g.groups = groups;
            g.nwin = nwin;
            g.wrows = wrows;
            g.lds = lds;
            // one round of workgroups
            g.chunks = std::max(1, 256 * per_cu / groups);
        }
    }
    if (best == 0.0) {
        g.lds = SIZE_MAX;
        return g;
    }
    g.rows = cdiv(cdiv(s.N, g.chunks), R) * R;
    g.chunks = cdiv(s.N, g.rows);
    return g;
}

struct FwdGeo {
    int nb, a, c, tasks, cmax, waves;
};

FwdGeo fwd_geo(const Shape &s, size_t budget) {
    FwdGeo f{};
    const int ks = ks_of(s.Q);
    f.nb = (int)cdiv(s.M, 16);
    f.a = fwd_a(ks);
    f.c = fwd_c(ks);
    const int full = f.a * f.c + 1;
    auto waves = [&](int cmax) {
        int n = 0;
        f.tasks = 0;
        for (int cb = 0; cb < f.nb; cb += f.c)
            for (int rb = cb; rb < f.nb; rb += f.a, ++f.tasks)
                n += fwd_chunks(s.N, f.nb, f.a, f.c, cb, rb, cmax);
        return n;
    };
    // the chunks with which the grid fills one round of two waves per SIMD, with the
    // partial sums within the region and at least kFwdMinRows rows in each
    const int64_t room = (int64_t)(budget / ((size_t)f.a * f.c * 256 * 8));
    const int64_t most = std::min<int64_t>(2 * kSimds, room);
    int64_t work = 0;   // full times the waves of cmax = 1, without the roundings
    for (int cb = 0; cb < f.nb; cb += f.c)
        for (int rb = cb; rb < f.nb; rb += f.a)
            work += fwd_tiles(f.nb, f.a, f.c, cb, rb) + 1;
    const int64_t cmax = std::min(most * full / work, cdiv(s.N, kFwdMinRows));
    f.cmax = (int)std::max<int64_t>(1, cmax);
    f.waves = waves(f.cmax);
    if (f.waves > room) f.cmax = 0;
    return f;
}

double *dbl(void *p, size_t off) { return reinterpret_cast<double *>(static_cast<char *>(p) + off); }

}  // namespace

bool f64_stats_wanted(const Shape &s) { return s.Q > 4 || (s.Q > 2 && s.M > 128); }
bool f64_grads_wanted(const Shape &s) { return s.Q > 2 || (s.Q > 1 && s.M > 128); }

size_t f64_region_bytes(const Shape &s) {
    size_t b = 0;
    if (f64_stats_wanted(s)) {
        const FwdGeo f = fwd_geo(s, SIZE_MAX);
        b = (size_t)f.waves * f.a * f.c * 256 * 8;
    }
    if (f64_grads_wanted(s)) b = std::max(b, f64_grad_plan(s, SIZE_MAX).end);
    return b;
}

bool f64_stats_fit(const Shape &s, size_t budget) {
    return f64_stats_wanted(s) && fwd_geo(s, budget).cmax >= 1;
}

hipError_t f64_psi2(const Shape &s, const double *mu, const double *Z, const double *w1,
                    const double *w2, const double *lp1, const double *lp2, const Hyp<double> &h,
                    double *psi0, double *Psi1, double *Psi2, int accumulate, void *ws, size_t budget,
                    hipStream_t st) {
    const FwdGeo f = fwd_geo(s, budget);
    double *partial = static_cast<double *>(ws);
    const unsigned grid = (unsigned)cdiv(f.waves, kFwdWaves);
    {
        TimedScope ts(st, "f64_psi2_fwd");
#define GPPS_F64_FWD(KS)                                                                          \
    case KS:                                                                                      \
        psi2_fwd_kernel<KS><<<grid, kFwdWaves * 64, 0, st>>>(s.N, (int)s.M, (int)s.Q, f.nb,        \
                                                             f.cmax, mu, Z, w2, lp2, partial);     \
        break
        switch (ks_of(s.Q)) {
            GPPS_F64_FWD(1); GPPS_F64_FWD(2); GPPS_F64_FWD(3); GPPS_F64_FWD(4); GPPS_F64_FWD(5);
            GPPS_F64_FWD(6); GPPS_F64_FWD(8); GPPS_F64_FWD(10); GPPS_F64_FWD(12); GPPS_F64_FWD(16);
            default: return hipErrorInvalidValue;
        }
#undef GPPS_F64_FWD
    }
    TimedScope ts(st, "f64_psi2_reduce_psi1");
    psi2_fwd_reduce_kernel<<<(unsigned)(f.tasks * f.a * f.c + psi1_grid(s.N, s.M, Psi1, 4096)), 256, 0, st>>>(
        s.N, (int)s.M, (int)s.Q, f.nb, f.a, f.c, f.cmax, f.tasks, partial, Z, h, psi0, Psi2, accumulate, mu,
        w1, lp1, Psi1);
    return hipGetLastError();
}

// Region: Gc = (G2 + G2^T)/2 o 2^C [Mp x Mp], row gradients [groups][2][N][Q] (only when groups > 1),
// dZ slabs [chunks][M][Q], row sums [chunks][groups][Q + 1].
F64GradPlan f64_grad_plan(const Shape &s, size_t budget) {
    F64GradPlan p{};
    if (!f64_grads_wanted(s)) return p;
    GradGeo g = grad_geo(s);
    if (g.lds > kLdsMax) return p;
    const int64_t Mp = cdiv(s.M, 16) * 16;
    size_t o = 0;
    auto take = [&](size_t n) { size_t r = o; o = align_up(o + n * 8, 256); return r; };
    p.off_gc = take(Mp * Mp);
    p.off_rowg = take(g.groups > 1 ? (size_t)g.groups * 2 * s.N * s.Q : 0);
    // as many chunks as the region has room for
    const size_t per = (size_t)(s.M * s.Q + g.groups * (s.Q + 1)) * 8;
    const int64_t room = budget > o + 512 ? (int64_t)((budget - o - 512) / per) : 0;
    if (room < 1) return p;  // ok = false
    if (g.chunks > room) {
        const int R = rows_of(ks_of(s.Q));
        g.rows = cdiv(cdiv(s.N, room), R) * R;
        g.chunks = cdiv(s.N, g.rows);
    }
    p.off_colp = take((size_t)g.chunks * s.M * s.Q);
    p.off_rowp = take((size_t)g.chunks * g.groups * (s.Q + 1));
    p.ok = o <= budget;
    p.end = o;
    p.chunks = g.chunks;
    p.rows = g.rows;
    p.groups = g.groups;
    p.nw = g.nw;
    p.wrows = g.wrows;
    p.nwin = g.nwin;
    p.lds = g.lds;
    return p;
}

hipError_t f64_psi2_grads(const Shape &s, const F64GradPlan &p, const double *mu, const double *S,
                          const double *Z, const double *w1, const double *w2, const double *lp1,
                          const double *lp2, const Hyp<double> &h, const double *G1,
                          const double *Gc, double *dmu, double *dS, void *ws, hipStream_t st) {
    const int nb = (int)cdiv(s.M, 16);
    // one group of columns writes dmu and dS themselves
    double *om = p.groups > 1 ? dbl(ws, p.off_rowg) : dmu;
    double *os = p.groups > 1 ? om + s.N * s.Q : dS;
    const dim3 grid((unsigned)p.groups, (unsigned)p.chunks);
    TimedScope ts(st, "f64_psi2_grad");
#define GPPS_F64_GRAD(KS)                                                                         \
    case KS: {                                                                                    \
        const hipError_t e = hipFuncSetAttribute((const void *)psi2_grad_kernel<KS>,              \
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,      \
                                                 (int)p.lds);                                     \
        if (e != hipSuccess) return e;                                                            \
        psi2_grad_kernel<KS><<<grid, p.nw * 64, p.lds, st>>>(                                     \
            s.N, (int)s.M, (int)s.Q, nb, p.wrows, p.nwin, p.rows, mu, S, Z, w1, w2, lp1, lp2, h,  \
            G1, Gc, om, os, dbl(ws, p.off_colp), dbl(ws, p.off_rowp));                            \
        break;                                                                                    \
    }
    switch (ks_of(s.Q)) {
        GPPS_F64_GRAD(1) GPPS_F64_GRAD(2) GPPS_F64_GRAD(3) GPPS_F64_GRAD(4) GPPS_F64_GRAD(5)
        GPPS_F64_GRAD(6) GPPS_F64_GRAD(8) GPPS_F64_GRAD(10) GPPS_F64_GRAD(12) GPPS_F64_GRAD(16)
        default: return hipErrorInvalidValue;
    }
#undef GPPS_F64_GRAD
    return hipGetLastError();
}

}  // namespace gpps
