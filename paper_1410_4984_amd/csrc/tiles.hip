// Psi2 and its gradients on the matrix instructions of the element type itself
// (v_mfma_f64_16x16x4f64, v_mfma_f64_4x4x4f64, v_mfma_f32_16x16x4f32): every operand,
// product and sum is double in fp64 and single in fp32.
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
// either.  The product is summed from zero and b_m + b_m' added last, so that its 4 k-steps
// round at half of the exponent's size or less: started from b_m + b_m' they left 2.7e-15
// of Psi2 in fp64 at Q = 30 (N = 200, M = 64), 1.2e-15 so (the vector kernels: 2.4e-15).
//
// What bounds these kernels is the SIMDs' issue rate.  In fp64 a 16 x 16 x 4 product
// occupies a SIMD for 64 cycles and no vector instruction issues meanwhile (measured: 8 FMAs
// behind each product add 8 FMAs' time), so matrix and vector work add up: a matrix FMA costs
// the same as a vector one, but needs one operand load per 16 of them, no cross-lane sums and
// no index arithmetic.  The exponential is 2^E' in 15 instructions (the table's
// ln 2 is folded into x and b), against about 21 of exp().  In fp32 a product takes 32
// cycles and the exponential is one instruction.
//
// Measured against the vector kernels before them (fp64, gradient + forward): 45.3 + 10.6 ms
// -> 15.1 + 5.0 ms at N = 100,000, M = 256, Q = 20, where the matrix cores are busy 46% of the
// gradient's cycles and 42% of the forward's and vector instructions 37% and 49%, never at
// once (SQ counters); 3.34 + 0.53 -> 1.46 + 0.49 ms at N = 50,000, M = 100, Q = 10; 261 + 3.7 ->
// 3.5 + 1.2 ms at N = 4096, M = 512, Q = 30.  fp32, statistics + gradients: 4.06 -> 1.65 ms
// at N = 3001, M = 700, Q = 12; 54 -> 0.67 ms at N = 1500, M = 300, Q = 40; 2.2 s -> 38 ms at
// N = 40,000, M = 700, Q = 31 (the vector kernels' z table did not fit LDS there).
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

constexpr size_t kLdsMax = 160 * 1024;
constexpr int kCus = 256, kSimds = 4 * kCus;
constexpr double kLog2e = 1.4426950408889634074;
// The largest |b| of the fast exponential (fp64: its integer part has to fit 32 bits;
// fp32: beyond it b's rounding passes 0.1, and 2^E' of such a row is zero).
template <typename T>
__host__ __device__ constexpr T slow_limit() { return sizeof(T) == 8 ? T(67108864.0) : T(1048576.0); }

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// The matrix instructions: 16 x 16 x 4 products (operand lane l holds row or column
// l % 16 and k = l / 16), whose result register v of lane group g holds row
// row(v, g), and, in fp64 only, four independent 4 x 4 x 4 ones.
template <typename T>
struct Mm;
template <>
struct Mm<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    static constexpr bool kFours = true;
    static __device__ v4 mul(double a, double b, v4 c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __host__ __device__ constexpr int row(int v, int g) { return 4 * v + g; }
};
template <>
struct Mm<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    static constexpr bool kFours = false;
    static __device__ v4 mul(float a, float b, v4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __host__ __device__ constexpr int row(int v, int g) { return 4 * g + v; }
};
__device__ inline double fours(double a, double b, double c) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}
template <typename T>
__device__ inline typename Mm<T>::v4 zero4() { return typename Mm<T>::v4{0, 0, 0, 0}; }
// Sum over the four lane groups (lanes l, l + 16, l + 32, l + 48), in every lane.
__device__ inline double sum_groups(double v) { return fours(1.0, v, 0.0); }
__device__ inline float sum_groups(float v) { return Mm<float>::mul(1.f, v, zero4<float>())[0]; }

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

__device__ inline float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline double dexp(double x) { return exp(x); }
__device__ inline float dexp(float x) { return __expf(x); }

// Psi2_n[m, m'] without the pair factor, by the closed form itself (slow rows).
template <typename T>
__device__ inline T direct_pair(const T *__restrict__ x, const T *__restrict__ w2, T lp2,
                                const T *__restrict__ za, const T *__restrict__ zb, int Q) {
    T e = lp2;
    for (int q = 0; q < Q; ++q) {
        const T d = x[q] - T(0.5) * (za[q] + zb[q]);
        e -= d * d * w2[q];
    }
    return dexp(e);
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
constexpr int64_t kFwdMaxFew = 8;   // chunks per task up to which more than one round is tried
constexpr int kFwdMinRows = 4;   // rows per chunk of the smallest calls (a row takes a wave 2 us alone)
constexpr int kFlush = 128;  // rows summed before they join the chunk's total (a multiple of grad_rows)

// Row and column blocks of a task.  Its z rows, x and sums fill the 256 registers of two waves
// per SIMD; in fp64 14 to 82 go to scratch from KS = 5 on (KS = 8: 82, 332 bytes a lane).
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
    return na * nc - (rb == cb && nc == 2 ? 1 : 0);   // C <= 2: one tile lies below the diagonal
}
// From the host: the row chunks of a task by its tiles (at most A C <= 8), and for each
// column group its first wave and its first task.
constexpr int kFwdGroups = GPPS_MAX_M / 16;
struct FwdTable {
    unsigned n[9];
    unsigned short wave0[kFwdGroups], task0[kFwdGroups];
};
// The last of `groups` (ascending) entries that is no more than x: every lane compares
// some of them (a search step by step took 20 us of a workgroup's life at M = 2000).
__device__ inline int last_group(const unsigned short *__restrict__ first, int groups, int x) {
    int n = 0;
    for (int i = 0; i < groups; i += 64) {
        const int k = i + (threadIdx.x & 63);
        n += __popcll(__ballot(k < groups && first[min(k, groups - 1)] <= x));
    }
    return __builtin_amdgcn_readfirstlane(n - 1);
}
// Of a column group's K tasks all but the first and the last have the same tiles:
// task k with its chunks and first wave.
__device__ inline FwdTask group_task(int nb, int A, int C, const FwdTable &n, int group, int k, int K) {
    const int cb = group * C, w0 = n.wave0[group];
    const int c0 = n.n[fwd_tiles(nb, A, C, cb, cb)];
    const int cm = K > 2 ? n.n[fwd_tiles(nb, A, C, cb, cb + A)] : 0;
    const int rb = cb + k * A;
    return FwdTask{cb, rb, w0 + (k == 0 ? 0 : c0 + (k - 1) * cm), (int)n.n[fwd_tiles(nb, A, C, cb, rb)]};
}
// The task that holds wave w of `waves`.
__device__ inline FwdTask fwd_task(int nb, int A, int C, const FwdTable &n, int w) {
    const int group = last_group(n.wave0, (nb + C - 1) / C, w), cb = group * C;
    const int K = (nb - cb + A - 1) / A;
    const int r = w - n.wave0[group] - (int)n.n[fwd_tiles(nb, A, C, cb, cb)];
    int k = 0;
    if (r >= 0) k = K > 2 ? min(1 + r / (int)n.n[fwd_tiles(nb, A, C, cb, cb + A)], K - 1) : 1;
    return group_task(nb, A, C, n, group, k, K);
}

template <typename T, int KS>
__global__ __launch_bounds__(kFwdWaves * 64, 2) void tiles_fwd_kernel(
    const int *__restrict__ gate, int64_t N, int M, int Q, int nb, int waves, FwdTable table, const T *__restrict__ mu,
    const T *__restrict__ Z, const T *__restrict__ w2, const T *__restrict__ lp2,
    T *__restrict__ partial) {
    if (gate && gate[0] == 0) return;
    using v4 = typename Mm<T>::v4;
    constexpr T kLog2 = T(kLog2e), kLim = T(0.25) * slow_limit<T>();
    constexpr int QP = 4 * KS, kFwdA = fwd_a(KS), kFwdC = fwd_c(KS), kFwdRows = fwd_rows(KS);
    __shared__ T t_mu[kFwdWaves][2][kFwdRows][QP], t_k[kFwdWaves][2][kFwdRows][QP],
        t_h[kFwdWaves][2][kFwdRows];
    const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto &s_mu = t_mu[wv];
    auto &s_k = t_k[wv];
    auto &s_h = t_h[wv];
    const int w = blockIdx.x * kFwdWaves + wv;
    if (w >= waves) return;
    const FwdTask task = fwd_task(nb, kFwdA, kFwdC, table, w);
    const int cb = task.cb, rb = task.rb, na = min(kFwdA, nb - rb);
    // blocks past the edge repeat the last inducing input (never stored)
    T za[kFwdA][KS], zc[kFwdC][KS];
#pragma unroll
    for (int a = 0; a < kFwdA; ++a) {
        const int m = min((rb + a) * 16 + c16, M - 1);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int q = 4 * s + g;
            const T v = Z[(int64_t)m * Q + min(q, Q - 1)];
            za[a][s] = q < Q ? v : T(0);
        }
    }
#pragma unroll
    for (int c = 0; c < kFwdC; ++c) {
        const int m = min((cb + c) * 16 + c16, M - 1);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int q = 4 * s + g;
            const T v = Z[(int64_t)m * Q + min(q, Q - 1)];
            zc[c][s] = q < Q ? v : T(0);
        }
    }
    v4 acc[kFwdA][kFwdC];
#pragma unroll
    for (int a = 0; a < kFwdA; ++a)
#pragma unroll
        for (int c = 0; c < kFwdC; ++c) acc[a][c] = zero4<T>();
    const int64_t r0 = N * (w - task.first) / task.chunks, r1 = N * (w - task.first + 1) / task.chunks;
    // partial[wave][tile][v][lane]
    T *out = partial + (int64_t)w * (kFwdA * kFwdC * 256) + lane;
    auto stage = [&](int64_t base, int buf) {
        const int cnt = (int)min<int64_t>(kFwdRows, r1 - base);
        for (int i = lane; i < kFwdRows * QP; i += 64) {
            const int r = i / QP, q = i - r * QP;
            const int64_t n = base + min(r, cnt - 1);
            const T m = mu[n * Q + min(q, Q - 1)], w = w2[n * Q + min(q, Q - 1)];
            s_mu[buf][r][q] = q < Q ? m : T(0);
            s_k[buf][r][q] = q < Q ? T(-0.5) * kLog2 * w : T(0);
        }
        if (lane < kFwdRows) s_h[buf][lane] = T(0.125) * kLog2 * lp2[base + min(lane, cnt - 1)];
    };
    int flushed = 0;
    if (r0 < r1) stage(r0, 0);
    int buf = 0;
    for (int64_t base = r0; base < r1; base += kFwdRows, buf ^= 1) {
        const int cnt = (int)min<int64_t>(kFwdRows, r1 - base);
        wave_lds_fence();
        if (base + kFwdRows < r1) stage(base + kFwdRows, buf ^ 1);
        for (int r = 0; r < cnt; ++r) {
            const T hl = s_h[buf][r];  // a quarter of lambda/2 lp2: one per lane group
            T muq[KS], kq[KS];
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                muq[s] = s_mu[buf][r][4 * s + g];
                kq[s] = s_k[buf][r][4 * s + g];
            }
            T x[kFwdC][KS], bc[kFwdC];
            bool ok = true;
#pragma unroll
            for (int c = 0; c < kFwdC; ++c) {
                T part = 0;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const T d = muq[s] - zc[c][s];
                    x[c][s] = kq[s] * d;
                    part = fma(x[c][s], d, part);
                }
                part = fma(T(0.5), part, hl);
                ok = ok && fabs(part) < kLim;
                bc[c] = sum_groups(part);
            }
#pragma unroll
            for (int a = 0; a < kFwdA; ++a) {
                if (a >= na) break;  // uniform
                __builtin_amdgcn_sched_barrier(0);
                T da[KS], part = 0;
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    da[s] = muq[s] - za[a][s];
                    part = fma(kq[s] * da[s], da[s], part);
                }
                part = fma(T(0.5), part, hl);
                if (__builtin_expect(__all(ok && fabs(part) < kLim), 1)) {
                    const v4 br = Mm<T>::mul(part, T(1), zero4<T>());
#pragma unroll
                    for (int c = 0; c < kFwdC; ++c) {
                        if (cb + c > rb + a || cb + c >= nb) break;  // uniform: below the diagonal
                        v4 e = zero4<T>();
#pragma unroll
                        for (int s = 0; s < KS; ++s) e = Mm<T>::mul(da[s], x[c][s], e);
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[a][c][v] += exp2_fast(e[v] + (br[v] + bc[c]));
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
                            const int mp = min((rb + a) * 16 + Mm<T>::row(v, l >> 4), M - 1);
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
        if (last || (base + kFwdRows - r0) % kFlush == 0) {
#pragma unroll
            for (int a = 0; a < kFwdA; ++a)
#pragma unroll
                for (int c = 0; c < kFwdC; ++c)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        T *o = out + ((a * kFwdC + c) * 4 + v) * 64;
                        *o = flushed ? *o + acc[a][c][v] : acc[a][c][v];
                        acc[a][c][v] = 0;
                    }
            flushed = 1;
        }
    }
}

// Workgroups of the reduce of `tasks` tasks: G to a tile, tiles in whole eights.
__host__ __device__ inline unsigned reduce_blocks(int tasks, int A, int C, int G) {
    return (unsigned)((tasks * A * C + 7) / 8 * 8 * G);
}
// Workgroups below those: Psi2[m, m'] = 2^C sum over chunks, both triangles and
// psi0.  256 / G entries of a task's tile each: thread group g of G takes chunks g,
// g + G, ... in order and the G sums are added in order.  G = 4 where a task has more than
// 16 chunks and 16 where it has more than 256: one thread per entry took 60 us for the
// 1,666 chunks of N = 30,000, M = 10, and 16 groups, whose reads are 64-byte pieces,
// 51 us instead of 20 for the 36 chunks of N = 300, M = 520.  The workgroups past them compute Psi1.
template <typename T>
__global__ __launch_bounds__(256) void tiles_reduce_kernel(
    const int *__restrict__ gate, int64_t N, int M, int Q, int nb, int A, int CB, FwdTable table,
    int tasks, int G, const T *__restrict__ partial, const T *__restrict__ Z, Hyp<T> h, T *__restrict__ psi0,
    T *__restrict__ Psi2, int accumulate, const T *__restrict__ mu, const T *__restrict__ w1,
    const T *__restrict__ lp1, T *__restrict__ Psi1) {
    if (gate && gate[0] == 0) return;
    __shared__ Psi1Lds<T> s_p1;
    __shared__ T s_sum[256];
    const unsigned rblocks = reduce_blocks(tasks, A, CB, G);
    if (blockIdx.x >= rblocks) {
        psi1_blocks<T>(s_p1, blockIdx.x - rblocks, gridDim.x - rblocks, N, M, Q, mu, Z, w1, lp1, Psi1,
                       [](T x) { return dexp(x); });
        return;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0)
        psi0[0] = (accumulate ? psi0[0] : T(0)) + (T)N * h.sf2;
    // the parts of a tile lie eight workgroups apart: they share cache lines of Psi2 (and
    // consecutive workgroups go to different XCDs)
    const int E = 256 / G, part = blockIdx.x / 8 % G, job = blockIdx.x / (8 * G) * 8 + blockIdx.x % 8;
    const int tile = job % (A * CB), number = job / (A * CB);
    if (number >= tasks) return;
    const int group = last_group(table.task0, (nb + CB - 1) / CB, number);
    const FwdTask task = group_task(nb, A, CB, table, group, number - table.task0[group],
                                    (nb - group * CB + A - 1) / A);
    const int cb = task.cb + tile % CB, rb = task.rb + tile / CB, chunks = task.chunks;
    if (cb >= nb || rb >= nb || cb > rb) return;
    const int g = threadIdx.x / E, entry = part * E + threadIdx.x % E;
    const int64_t stride = A * CB * 256;
    const T *src = partial + task.first * stride + tile * 256 + entry;
    // eight loads in flight together, from clamped addresses past the last chunk
    T s = 0;
    for (int k = g; k < chunks; k += 8 * G) {
        T t[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = src[min(k + j * G, chunks - 1) * stride];
#pragma unroll
        for (int j = 0; j < 8; ++j) s += k + j * G < chunks ? t[j] : T(0);
    }
    if (G > 1) {
        s_sum[threadIdx.x] = s;
        __syncthreads();
        if (g != 0) return;
        s = 0;
        for (int j = 0; j < G; ++j) s += s_sum[j * E + threadIdx.x];
    }
    const int lane = entry & 63, v = entry >> 6;
    const int m = cb * 16 + (lane & 15), mp = rb * 16 + Mm<T>::row(v, lane >> 4);
    if (m >= M || mp >= M || m > mp) return;
    T C = 0;
#pragma unroll 8
    for (int q = 0; q < Q; ++q) {
        const T dz = Z[(int64_t)m * Q + q] - Z[(int64_t)mp * Q + q];
        C -= dz * dz / (T(4) * h.l2[q]);
    }
    const T val = (accumulate ? Psi2[(int64_t)m * M + mp] : T(0)) + dexp(C) * s;
    Psi2[(int64_t)m * M + mp] = val;
    Psi2[(int64_t)mp * M + m] = val;
}

// ---------------------------------------------------------------- gradient
template <int CTRL>
__device__ inline float rotate16(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ inline double rotate16(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// Sums within the 16 lanes of a lane group: over the lanes of equal lane & 3, and
// over all of them; in every lane.
template <typename T>
__device__ inline T sum_fours(T v) {
    v += rotate16<0x128>(v);  // row_ror:8
    v += rotate16<0x124>(v);
    return v;
}
template <typename T>
__device__ inline T sum16(T v) {
    v = sum_fours(v);
    v += rotate16<0x122>(v);
    v += rotate16<0x121>(v);
    return v;
}

// Rows n a wave works on at once: each serves the same z and Gc operands again, and keeps x, U
// and its row values for 2 column blocks in registers.  Two where that measured faster than one
// (fp64: 15.6 ms with two and 15.0 with one at Q = 20; fp32 would hold four up to Q = 16: 5%
// faster at M >= 700, 5-70% slower below).
constexpr int grad_rows(int ks, size_t elem) { return ks <= (elem == 8 ? 4 : 12) ? 2 : 1; }

// The reference c of a row's second product: where a Gaussian with the centre and variance of
// Z, weighted by the row's (mu, 1 / w2), has its mean.  Near the centre where Z spreads
// less than the row sees, near mu where it spreads more; mu where that is not finite.
template <typename T>
__device__ inline T reference(T mu, T w2, T centre, T var) {
    const T s = var * w2, c = centre + (mu - centre) * (s / (T(1) + s));
    return fabs(c) <= T(1e38) ? c : mu;
}

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
// the generic pairs kernel).  dZ and dl take n_m = d_m r_m - V_m = sum_m' W (z_m' - z_m),
// of the size of the spacing of the Z whose W matters, while d r and V are of that of
// d: where S >> l^2 their difference loses sqrt(l^2 + 2 S) / l of its precision.  So the
// second product is U_m = sum_{m' != m} W (z_m' - c) with a reference c per row and
// dimension that is near those Z (reference()), and n = U - (z_m - c) (r - W[m, m]),
// d r + V = 2 d r - n.  The pair (m, m), which adds nothing to n, stays out of U and of
// its r: where Z is spread over many lengthscales it is most of r.  Against the difference
// of d r and V (long-double reference, S in 0.5 .. 2, N = 300, M = 64, relative error of dl):
// Q = 10, l = 0.005, Z within l: fp32 2.7e-4 -> 4.4e-6, fp64 6.5e-13 -> 2.4e-14; Q = 12,
// l = 0.002: 4.6e-4 -> 2.3e-6, 7.9e-13 -> 1.3e-14; Q = 10, l = 0.05, Z spread over 20 l in
// groups of neighbours: 1.5e-5 -> 1.6e-6, 3.2e-14 -> 2.4e-14.  It costs 1-8% of the
// gradients' time up to Q = 48 (fp64 14.8 -> 15.0 ms at N = 100,000, M = 256, Q = 20; fp32
// 1.20 -> 1.23 ms at N = 3,001, M = 700, Q = 12) and 12% past it in fp64.
// A wave owns 32 columns m and walks the blocks of
// 16 rows m': a tile of W leaves the exponent's product in exactly the layout
// that the second product, U^T += (z - c)^T W, takes as its right operand, and U comes
// out in the layout of x, so neither goes through LDS.  Each (m', z, Gc) operand
// serves 2 R products.  r is summed on the vector unit: 4 additions a tile, where a
// column of ones would cost 64 cycles.  Sums over m (dmu, dS, dl) go through the
// lanes and then the waves in a fixed order; dZ stays in LDS slots that one lane
// owns, for kFlush rows at a time: a chunk of N = 40,000, M = 2048 has 1,250 rows, and where
// these are alike their sum in one go left 323 2^-24 of dZ in fp32, 35 2^-24 so.
template <typename T, int KS>
__global__ __launch_bounds__(512) void tiles_grad_kernel(
    const int *__restrict__ gate, int64_t N, int M, int Q, int nb, int wrows, int nwin, int64_t rows_per_chunk,
    const T *__restrict__ mu, const T *__restrict__ S, const T *__restrict__ Z,
    const T *__restrict__ w1t, const T *__restrict__ w2t, const T *__restrict__ lp1,
    const T *__restrict__ lp2, Hyp<T> h, const T *__restrict__ G1,
    const T *__restrict__ Gc, const T *__restrict__ zref, T *__restrict__ dmu, T *__restrict__ dS,
    T *__restrict__ colpart, T *__restrict__ rowpart) {
    if (gate && gate[0] == 0) return;
    using v4 = typename Mm<T>::v4;
    constexpr T kLog2 = T(kLog2e), kLim = slow_limit<T>();
    // T16 tiles of 16 dimensions and T4 of 4 hold U; QP: that width (zero past Q)
    constexpr int T16 = Mm<T>::kFours ? KS / 4 : (KS + 3) / 4, T4 = Mm<T>::kFours ? KS % 4 : 0;
    constexpr int NT = T16 + T4, QP = 16 * T16 + 4 * T4, QK = 4 * KS, ZS = QP + 1, R = grad_rows(KS, sizeof(T));
    constexpr int RV = 5;                // values staged for a row and dimension
    extern __shared__ double sm_[];
    T *sm = reinterpret_cast<T *>(sm_);
    const int tid = threadIdx.x, nthr = blockDim.x, nw = nthr >> 6;
    const int lane = tid & 63, g = lane >> 4, c16 = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wcols = nw * kGradC * 16;
    T *sz = sm;                          // [wrows][ZS]
    T *sb = sz + wrows * ZS;             // [R][wrows]: b of the rows, permuted in each block
    T *sbc = sb + R * wrows;             // [R][wcols]: b of the workgroup's columns
    T *srow = sbc + R * wcols;           // [R][RV][QP]: mu, w1, w2, S, c
    T *slp = srow + R * RV * QP;         // [R][2]: lp1, lp2
    T *sred = slp + R * 2;               // [nw][R][3 QP + 2]
    T *sdl = sred + nw * R * (3 * QP + 2);  // [R][QP + 1]
    T *shyp = sdl + R * (QP + 1);        // [3][QP]: 1/l^2, l, 1/l^3
    T *sgz = shyp + 3 * QP;              // [wcols][QP]
    int *sslow = reinterpret_cast<int *>(sgz + wcols * QP);  // [2][R]
    const int Mp = nb * 16;
    const int cb0 = (blockIdx.x * nw + wv) * kGradC;       // the wave's first column block
    const int ncol = min(kGradC, nb - cb0);                // its column blocks (<= 0: none)
    const int m0 = blockIdx.x * wcols;                     // the workgroup's first column
    for (int q = tid; q < QP; q += nthr) {
        const T l = q < Q ? h.l[q] : T(1.0), l2 = q < Q ? h.l2[q] : T(1.0);
        shyp[q] = T(1.0) / l2;
        shyp[QP + q] = l;
        shyp[2 * QP + q] = T(1.0) / (l2 * l);
    }
    for (int i = tid; i < R * (QP + 1); i += nthr) sdl[i] = T(0.0);
    for (int i = tid; i < wcols * QP; i += nthr) sgz[i] = T(0.0);
    // rows of Z past M repeat the last one: finite wherever the real ones are
    auto stage_z = [&](int w0) {
        for (int i = tid; i < wrows * QP; i += nthr) {
            const int r = i / QP, q = i - r * QP;
            const T v = Z[(int64_t)min(w0 + r, M - 1) * Q + min(q, Q - 1)];
            sz[r * ZS + q] = q < Q ? v : T(0.0);
        }
    };
    if (nwin == 1) stage_z(0);
    // coordinate q of inducing input m (any q where the row values are zero beyond Q)
    auto zcol = [&](int m, int q) {
        return nwin == 1 ? sz[m * ZS + q] : Z[(int64_t)m * Q + min(q, Q - 1)];
    };
    const int64_t r0 = (int64_t)blockIdx.y * rows_per_chunk, r1 = min(N, r0 + rows_per_chunk);
    bool flushed = false;
    for (int64_t base = r0; base < r1; base += R) {
        const int cnt = (int)min<int64_t>(R, r1 - base);
        __syncthreads();
        for (int i = tid; i < R * RV * QP; i += nthr) {
            const int r = i / (RV * QP), k = i / QP - r * RV, q = i % QP, qc = min(q, Q - 1);
            const int64_t j = (base + min(r, cnt - 1)) * Q + qc;
            const T *src = k == 1 ? w1t : k == 2 ? w2t : k == 3 ? S : mu;
            T v = src[j];
            if (k == 4 && Gc) v = reference(v, w2t[j], zref[qc], zref[Q + qc]);
            srow[i] = q < Q ? v : T(0.0);
        }
        if (tid < R) {
            slp[2 * tid] = lp1[base + min(tid, cnt - 1)];
            slp[2 * tid + 1] = lp2[base + min(tid, cnt - 1)];
        }
        if (tid < 2 * R) sslow[tid] = 0;
        __syncthreads();
        // sum over q of w (x - z)^2, w the row's w1 or w2, as two sums side by side (rounding)
        auto squares = [&](int r, int which, auto z) {
            const T *xr = srow + r * RV * QP, *w = xr + which * QP;
            T s[2] = {0, 0};
#pragma unroll 2
            for (int q = 0; q < QK / 2; ++q)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const T d = xr[2 * q + j] - z(2 * q + j);
                    s[j] = fma(w[2 * q + j] * d, d, s[j]);
                }
            return s[0] + s[1];
        };
        // b of row r and an inducing input
        auto b_of = [&](int r, auto z) {
            return kLog2 * (T(0.5) * slp[2 * r + 1] - T(0.25) * squares(r, 2, z));
        };
        // place of row j in sb: row(v, g) of a block at 4 g + v, so that a lane's four
        // are contiguous
        auto b_at = [](int j) {
            return Mm<T>::row(1, 0) == 4 ? (j & ~15) + 4 * (j & 3) + ((j >> 2) & 3) : j;
        };
        if (nwin > 1)  // else the columns are among the rows of the one window
            for (int i = tid; i < R * wcols; i += nthr) {
                const int r = i / wcols;
                const T *z = Z + (int64_t)min(m0 + i - r * wcols, M - 1) * Q;
                const T s = b_of(r, [&](int q) { return z[min(q, Q - 1)]; });
                sbc[i] = s;
                if (!(fabs(s) < kLim)) sslow[r] = 1;
            }
        T x[R][kGradC][KS], rs[R][kGradC], rd[R][kGradC];   // rs: sums of W over m' != m, rd: W[m, m]
        v4 U16[R][kGradC][T16 > 0 ? T16 : 1];
        T U4[R][kGradC][T4 > 0 ? T4 : 1];
        // the Psi1 terms t = dL/dPsi1 o Psi1: lane l has rows 2 u + l / 32, column l % 32
        T tval[(R + 1) / 2];
#pragma unroll
        for (int u = 0; u < (R + 1) / 2; ++u) {
            tval[u] = 0;
            const int r = 2 * u + (lane >> 5), m = cb0 * 16 + (lane & 31);
            if (G1 && r < cnt && m < M)
                tval[u] = G1[(base + r) * M + m] *
                          dexp(slp[2 * r] - T(0.5) * squares(r, 1, [&](int q) { return zcol(m, q); }));
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < kGradC; ++c) {
                rs[r][c] = rd[r][c] = T(0.0);
                const int m = min((cb0 + c) * 16 + c16, M - 1);
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const int q = 4 * s + g;
                    const T d = srow[r * RV * QP + q] - zcol(m, q);
                    x[r][c][s] = -T(0.5) * kLog2 * srow[r * RV * QP + 2 * QP + q] * d;
                }
#pragma unroll
                for (int t = 0; t < T16; ++t) U16[r][c][t] = zero4<T>();
#pragma unroll
                for (int t = 0; t < T4; ++t) U4[r][c][t] = T(0.0);
            }
        if (Gc) {
            T bi[R][kGradC];
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
                    const T s = b_of(r, [&](int q) { return sz[j * ZS + q]; });
                    sb[r * wrows + b_at(j)] = s;
                    if (!(fabs(s) < kLim)) sslow[R + r] = 1;
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
                T muA[R][KS], cB[R][NT];
#pragma unroll
                for (int r = 0; r < R; ++r) {
#pragma unroll
                    for (int s = 0; s < KS; ++s) muA[r][s] = srow[r * RV * QP + 4 * s + g];
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        cB[r][t] = srow[(r * RV + 4) * QP + (t < T16 ? 16 * t + c16
                                                                     : 16 * T16 + 4 * (t - T16) + (lane & 3))];
                }
                const int jn = min(wrows, Mp - w0) / 16;
                // NC: the wave's column blocks, so that their tiles interleave
                auto tiles = [&](auto ncc) {
                    constexpr int NC = decltype(ncc)::value;
                    for (int J = 0; J < jn; ++J) {
                        T G[NC][4];
#pragma unroll
                        for (int c = 0; c < NC; ++c)
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                G[c][v] = Gc[(int64_t)(w0 + 16 * J + Mm<T>::row(v, g)) * Mp + (cb0 + c) * 16 + c16];
                        T zA[KS];
#pragma unroll
                        for (int s = 0; s < KS; ++s) zA[s] = sz[(16 * J + c16) * ZS + 4 * s + g];
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            __builtin_amdgcn_sched_barrier(0);
                            T W[NC][4];
                            if (__builtin_expect(!slow[r], 1)) {
                                T dA[KS];
                                v4 e[NC];
#pragma unroll
                                for (int c = 0; c < NC; ++c) e[c] = zero4<T>();
#pragma unroll
                                for (int s = 0; s < KS; ++s) dA[s] = muA[r][s] - zA[s];
#pragma unroll
                                for (int s = 0; s < KS; ++s)
#pragma unroll
                                    for (int c = 0; c < NC; ++c) e[c] = Mm<T>::mul(dA[s], x[r][c][s], e[c]);
#pragma unroll
                                for (int c = 0; c < NC; ++c)
#pragma unroll
                                    for (int v = 0; v < 4; ++v) {
                                        const T b = sb[r * wrows + 16 * J + 4 * g + v] + bi[r][c];
                                        W[c][v] = G[c][v] * exp2_fast(e[c][v] + b);
                                    }
                            } else {
                                int l = lane;  // opaque: nothing of this branch is kept outside it
                                asm volatile("" : "+v"(l));
#pragma unroll
                                for (int c = 0; c < NC; ++c)
#pragma unroll
                                    for (int v = 0; v < 4; ++v) {
                                        const int m = (cb0 + c) * 16 + (l & 15);
                                        const int mp = w0 + 16 * J + Mm<T>::row(v, l >> 4);
                                        __builtin_amdgcn_sched_barrier(0);
                                        W[c][v] = T(0.0);
                                        if (m < M && mp < M)
                                            W[c][v] = G[c][v] *
                                                      direct_pair(srow + r * RV * QP,
                                                                  srow + r * RV * QP + 2 * QP,
                                                                  slp[2 * r + 1], Z + (int64_t)m * Q,
                                                                  Z + (int64_t)mp * Q, Q);
                                    }
                            }
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int c = 0; c < NC; ++c)
                                if (__builtin_expect(w0 + 16 * J == (cb0 + c) * 16, 0)) {  // uniform: on the diagonal
#pragma unroll
                                    for (int v = 0; v < 4; ++v)
                                        if (Mm<T>::row(v, g) == c16) {
                                            rd[r][c] = W[c][v];
                                            W[c][v] = T(0.0);
                                        }
                                }
#pragma unroll
                            for (int c = 0; c < NC; ++c)
                                rs[r][c] += (W[c][0] + W[c][1]) + (W[c][2] + W[c][3]);
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                T uB[NT];
#pragma unroll
                                for (int t = 0; t < NT; ++t)
                                    uB[t] = sz[(16 * J + Mm<T>::row(v, g)) * ZS +
                                               (t < T16 ? 16 * t + c16 : 16 * T16 + 4 * (t - T16) + (lane & 3))] -
                                            cB[r][t];
#pragma unroll
                                for (int c = 0; c < NC; ++c) {
#pragma unroll
                                    for (int t = 0; t < T16; ++t)
                                        U16[r][c][t] = Mm<T>::mul(W[c][v], uB[t], U16[r][c][t]);
#pragma unroll
                                    for (int t = 0; t < T4; ++t)
                                        U4[r][c][t] = fours(W[c][v], uB[T16 + t], U4[r][c][t]);
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
        // epilogue: of a 16-wide tile t lane (g, c16) holds (m = row(v, g),
        // q = 16 t + c16), of a 4-wide one (m = (lane & 12) + g, q = 16 T16 + 4 t + (lane & 3))
        if (ncol > 0) {
            int le = lane;  // opaque: the epilogue's addresses are formed here, not kept over the tiles
            asm volatile("" : "+v"(le));
            const int ge = le >> 4, ce = le & 15;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (r >= cnt) break;  // uniform
                T *red = sred + (wv * R + r) * (3 * QP + 2);
                v4 r16[kGradC], dm16[kGradC];
                T r4[kGradC], dm4[kGradC], rt = T(0.0), tt = T(0.0);
#pragma unroll
                for (int c = 0; c < kGradC; ++c) {
                    if (c >= ncol) rs[r][c] = rd[r][c] = T(0.0);
                    rt += rs[r][c] + rd[r][c];
                    tt += __shfl(tval[r / 2], 32 * (r & 1) + 16 * c + ce);
                    if (T16 > 0) r16[c] = Mm<T>::mul(rs[r][c], T(1.0), zero4<T>());
                    if (T4 > 0) r4[c] = fours(rs[r][c], T(1.0), T(0.0));
                    if (T16 > 0) dm16[c] = Mm<T>::mul(rd[r][c], T(1.0), zero4<T>());
                    if (T4 > 0) dm4[c] = fours(rd[r][c], T(1.0), T(0.0));
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
                    const T *row = srow + r * RV * QP + q;
                    const T xm = row[0], a1 = row[QP], a2 = row[2 * QP], cq = row[4 * QP];
                    const T il2 = shyp[q], l = shyp[QP + q], il3 = shyp[2 * QP + q];
                    T sp0 = T(0.0), st0 = T(0.0), su = T(0.0), sn = T(0.0), sx = T(0.0);
#pragma unroll
                    for (int c = 0; c < kGradC; ++c) {
                        if (c >= ncol) break;  // uniform
#pragma unroll
                        for (int v = 0; v < (wide ? 4 : 1); ++v) {
                            const int ml = wide ? Mm<T>::row(v, ge) : (le & 12) + ge;
                            const int m = min((cb0 + c) * 16 + ml, M - 1);
                            const T rm = wide ? r16[c][v] : r4[c];
                            const T tm = __shfl(tval[r / 2], 32 * (r & 1) + 16 * c + ml);
                            const T U = wide ? U16[r][c][wide ? t : 0][v] : U4[r][c][wide ? 0 : t - T16];
                            const T rmm = wide ? dm16[c][v] : dm4[c];
                            const T z = zcol(m, q), d = xm - z, dr = d * (rm + rmm), td = tm * d;
                            const T n = fma(cq - z, rm, U), p = T(2.0) * dr - n;
                            sp0 += dr;
                            st0 += td;
                            su = fma(d, p, su);
                            sn = fma(d, n, sn);
                            sx = fma(d, td, sx);
                            T *gz = sgz + ((wv * kGradC + c) * 16 + ml) * QP + q;
                            *gz += fma(a2, p, fma(il2, n, a1 * td));
                        }
                    }
                    const T u = a2 * a2 * su, y = a1 * a1 * sx;
                    T v0 = sum_groups(-T(2.0) * a2 * sp0 - a1 * st0);
                    T v1 = sum_groups(u + T(0.5) * y);
                    T v2 = sum_groups(fma(sn, il3, l * (u + y)));
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
            T v0 = T(0.0), v1 = T(0.0), v2 = T(0.0), Rt = T(0.0), Tt = T(0.0);
            for (int w = 0; w < live; ++w) {
                const T *red = sred + (w * R + r) * (3 * QP + 2);
                v0 += red[q];
                v1 += red[QP + q];
                v2 += red[2 * QP + q];
                Rt += red[3 * QP];
                Tt += red[3 * QP + 1];
            }
            const T *row = srow + r * RV * QP + q;
            const T a1 = row[QP], a2 = row[2 * QP], sv = row[3 * QP], il = T(1.0) / shyp[QP + q];
            const int64_t o = ((int64_t)blockIdx.x * 2 * N + base + r) * Q + q;
            dmu[o] = v0;
            dS[o] = v1 - a2 * Rt - T(0.5) * a1 * Tt;
            sdl[r * (QP + 1) + q] += v2 + (T(2.0) * sv * a2 * il) * Rt + (sv * a1 * il) * Tt;
            if (q == 0) sdl[r * (QP + 1) + QP] += T(2.0) * Rt + Tt;
        }
        // two-level sums, as in the forward: kFlush rows, then into the chunk's totals in HBM
        if (base + R >= r1 || (base + R - r0) % kFlush == 0) {
            __syncthreads();
            for (int i = tid; i < wcols * Q; i += nthr) {
                const int cc = i / Q, q = i - cc * Q;
                if (m0 + cc >= M) continue;
                T *o = colpart + ((int64_t)blockIdx.y * M + m0 + cc) * Q + q;
                *o = flushed ? *o + sgz[cc * QP + q] : sgz[cc * QP + q];
                sgz[cc * QP + q] = T(0.0);
            }
            for (int q = tid; q <= Q; q += nthr) {
                T s = T(0.0);
                for (int r = 0; r < R; ++r) {
                    T *v = sdl + r * (QP + 1) + (q < Q ? q : QP);
                    s += *v;
                    *v = T(0.0);
                }
                if (q == Q) s /= h.sf2;
                T *o = rowpart + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * (Q + 1) + q;
                *o = flushed ? *o + s : s;
            }
            flushed = true;
        }
    }
}

// k-steps of 4 dimensions, rounded to the instantiated widths
int ks_of(int64_t Q) {
    for (int ks : {1, 2, 3, 4, 5, 6, 8, 10, 12})
        if (Q <= 4 * ks) return ks;
    return 16;
}

size_t grad_lds(int ks, int nw, int wrows, size_t elem) {
    // as in the kernel: fp32 U comes in tiles of 16 dimensions only
    const int QP = elem == 8 ? 4 * ks : (ks + 3) / 4 * 16, R = grad_rows(ks, elem), wcols = nw * kGradC * 16;
    const size_t d = (size_t)wrows * (QP + 1) + R * wrows + R * wcols + R * 5 * QP + R * 2 +
                     (size_t)nw * R * (3 * QP + 2) + R * (QP + 1) + 3 * QP + (size_t)wcols * QP;
    return align_up(d * elem, 8) + 2 * R * 4 + 8;
}


GradGeo grad_geo(const Shape &s, size_t elem) {
    GradGeo g{};
    const int ks = ks_of(s.Q), R = grad_rows(ks, elem);
    const int nb = (int)cdiv(s.M, 16), need = (int)cdiv(nb, kGradC);  // waves per row chunk
    // the waves per workgroup that keep the most of a CU's eight wave slots (two per
    // SIMD: the register limit) on column blocks that exist, in at most one group of
    // columns per 128 (each writes dmu and dS of its own); the widest of equal ones.
    // fp32 up to Q = 16 has three waves per SIMD: 11% faster at M <= 256, but 30% slower
    // at M = 520 and 700, whose workgroups then hold fewer columns
    const int slots = elem == 4 && ks <= 4 && s.M <= 256 ? 12 : 8;
    double best = 0.0;
    for (int nw = std::min(8, need); nw >= 1; --nw) {
        const int groups = (int)cdiv(need, nw);
        if (groups > cdiv(nb, 8)) break;
        // Z whole in LDS where it fits, else the fewest equal windows that do
        int nwin = 1, wrows;
        size_t lds;
        for (;; ++nwin) {
            wrows = (int)cdiv(nb, nwin) * 16;
            lds = grad_lds(ks, nw, wrows, elem);
            if (lds <= kLdsMax || wrows == 16) break;
        }
        if (lds > kLdsMax) continue;
        const int per_cu = (int)std::min<int64_t>((int64_t)(kLdsMax / lds), slots / nw);
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
    g.rows = cdiv(cdiv(s.N, g.chunks), R) * R;
    g.chunks = cdiv(s.N, g.rows);
    return g;
}

struct FwdGeo {
    int nb, a, c, tasks, cmax, waves;
    FwdTable table;
};

// more: chunks past one round of workgroups, where the region has room for them.
FwdGeo fwd_geo(const Shape &s, size_t budget, size_t elem, bool more) {
    FwdGeo f{};
    const int ks = ks_of(s.Q);
    f.nb = (int)cdiv(s.M, 16);
    f.a = fwd_a(ks);
    f.c = fwd_c(ks);
    const int full = f.a * f.c + 1;
    // over the tasks: of a column group all but the first and last have the same tiles
    auto each = [&](auto fn) {
        for (int cb = 0; cb < f.nb; cb += f.c) {
            const int k = (f.nb - cb + f.a - 1) / f.a;
            fn(cb, cb, 1);
            if (k > 2) fn(cb, cb + f.a, k - 2);
            if (k > 1) fn(cb, cb + (k - 1) * f.a, 1);
        }
    };
    // the chunks with which the grid fills one round of two or three waves per SIMD, with the
    // partial sums within the region and at least kFwdMinRows rows in each
    const int64_t room = (int64_t)(budget / ((size_t)f.a * f.c * 256 * elem));
    // waves per SIMD: by the register count, and the LDS of the staged rows
    const int per_simd = elem == 4 && ks <= 6 ? 3 : 2;
    const int64_t most = std::min<int64_t>(per_simd * kSimds, room);
    // ceil(cmax (t + 1) / full) chunks for a task of t tiles, so that none takes longer than
    // a full one (rounded down, the diagonal's seven-tile tasks took a third longer at M = 2000)
    int64_t work = 0;   // full times the waves of cmax = 1, without the roundings
    each([&](int cb, int rb, int n) {
        work += (int64_t)n * (fwd_tiles(f.nb, f.a, f.c, cb, rb) + 1);
        f.tasks += n;
    });
    auto plan = [&](int64_t cmax) {
        f.cmax = (int)cmax;
        for (int t = 0; t <= 8; ++t) f.table.n[t] = (unsigned)std::min(s.N, cdiv(cmax * (t + 1), full));
        f.waves = 0;
        each([&](int cb, int rb, int n) {
            f.waves += n * f.table.n[fwd_tiles(f.nb, f.a, f.c, cb, rb)];
        });
    };
    const int64_t rows = cdiv(s.N, kFwdMinRows);
    int64_t cmax = std::max<int64_t>(1, std::min(most * full / work, rows));
    for (plan(cmax); f.waves > most && cmax > 1; plan(--cmax)) {}
    // From about M = 1000 on one round is a few chunks per task, and the workgroups (a wave on
    // every SIMD of a CU) that fill no whole round leave most CUs idle: 264 at M = 2048 in fp64
    // take as long as 512 would.  Up to kFwdMaxFew chunks, then, as many as bring the CUs'
    // largest share of the rows, workgroups per CU / chunks, within 3% of its least (fp64,
    // N = 6,000: at M = 2048 25.1 -> 13.7 ms for Q = 5 and 22.2 -> 12.2 for Q = 3, the vector
    // kernels 19.9 and 15.5; at M = 3000, Q = 3 33.9 -> 23.3, the vector kernels 30.2).
    if (more && cmax < kFwdMaxFew) {
        auto share = [&] { return (double)cdiv(cdiv(f.waves, kFwdWaves), kCus) / f.cmax; };
        double least = share();
        const int64_t last = std::min(kFwdMaxFew, rows);
        auto fits = [&] { return f.waves <= std::min<int64_t>(room, 65536); };   // 16-bit wave numbers
        for (int64_t c = cmax + 1; c <= last; ++c) {
            plan(c);
            if (fits()) least = std::min(least, share());
        }
        for (plan(cmax); f.cmax < last && !(fits() && share() <= 1.03 * least); plan(f.cmax + 1)) {}
        if (!fits()) plan(cmax);
    }
    int wave = 0, task = 0;
    each([&](int cb, int rb, int n) {
        if (rb == cb) {
            f.table.wave0[cb / f.c] = (unsigned short)wave;
            f.table.task0[cb / f.c] = (unsigned short)task;
        }
        wave += n * f.table.n[fwd_tiles(f.nb, f.a, f.c, cb, rb)];
        task += n;
    });
    return f;
}

template <typename T>
T *at(void *p, size_t off) { return reinterpret_cast<T *>(static_cast<char *>(p) + off); }

}  // namespace

bool tiles_stats_wanted(const Shape &s, size_t elem) {
    return s.Q > 4 || (elem == 8 && s.Q > 2 && s.M > 128);
}
bool tiles_grads_wanted(const Shape &s, size_t elem) {
    if (s.Q <= 2 || s.Q > 4) return s.Q > 4;
    return elem == 8 || (s.M > 170 && s.M <= 384) || s.M > 512;
}

TilesRegion tiles_region(const Shape &s, size_t elem) {
    TilesRegion r{0, 0};
    if (tiles_stats_wanted(s, elem)) {
        const FwdGeo f = fwd_geo(s, SIZE_MAX, elem, false);
        const size_t per = (size_t)f.a * f.c * 256 * elem;
        r.least = f.tasks * per;
        r.want = f.waves * per;
    }
    if (tiles_grads_wanted(s, elem)) {
        const TilesGradPlan g = tiles_grad_plan(s, SIZE_MAX, elem);
        // of the chunks' slabs one is needed
        r.want = std::max(r.want, g.end);
        r.least = std::max(r.least, g.off_colp + align_up(elem * s.M * s.Q, 256) +
                                        align_up(elem * g.groups * (s.Q + 1), 256) + 1024);
    }
    return r;
}

template <typename T>
hipError_t tiles_psi2(const Shape &s, const T *mu, const T *Z, const T *w1, const T *w2, const T *lp1,
                      const T *lp2, const Hyp<T> &h, T *psi0, T *Psi1, T *Psi2, int accumulate, void *ws,
                      size_t budget, const int *gate, hipStream_t st) {
    const FwdGeo f = fwd_geo(s, budget, sizeof(T), true);
    T *partial = static_cast<T *>(ws);
    const unsigned grid = (unsigned)cdiv(f.waves, kFwdWaves);
    {
        TimedScope ts(st, "tiles_psi2_fwd");
#define GPPS_TILES_FWD(KS)                                                                        \
    case KS:                                                                                      \
        if constexpr (KS > 1 || sizeof(T) == 8) /* fp32 comes here from Q = 5 on */               \
            tiles_fwd_kernel<T, KS><<<grid, kFwdWaves * 64, 0, st>>>(                             \
                gate, s.N, (int)s.M, (int)s.Q, f.nb, f.waves, f.table, mu, Z, w2, lp2, partial);  \
        break
        switch (ks_of(s.Q)) {
            GPPS_TILES_FWD(1); GPPS_TILES_FWD(2); GPPS_TILES_FWD(3); GPPS_TILES_FWD(4);
            GPPS_TILES_FWD(5); GPPS_TILES_FWD(6); GPPS_TILES_FWD(8); GPPS_TILES_FWD(10);
            GPPS_TILES_FWD(12); GPPS_TILES_FWD(16);
            default: return hipErrorInvalidValue;
        }
#undef GPPS_TILES_FWD
    }
    const int G = f.cmax > 256 ? 16 : f.cmax > 16 ? 4 : 1;
    TimedScope ts(st, "tiles_psi2_reduce_psi1");
    tiles_reduce_kernel<T><<<reduce_blocks(f.tasks, f.a, f.c, G) + psi1_grid(s.N, s.M, Psi1, gate ? 2048 : 4096),
                             256, 0, st>>>(gate, s.N, (int)s.M, (int)s.Q, f.nb, f.a, f.c, f.table, f.tasks, G,
                                           partial, Z, h, psi0, Psi2, accumulate, mu, w1, lp1, Psi1);
    return hipGetLastError();
}

// Region: Gc = (G2 + G2^T)/2 o 2^C [Mp x Mp], centre and variance of Z [2][Q], row gradients
// [groups][2][N][Q] (only when groups > 1), dZ slabs [chunks][M][Q], row sums [chunks][groups][Q + 1].
TilesGradPlan tiles_grad_plan(const Shape &s, size_t budget, size_t elem) {
    TilesGradPlan p{};
    GradGeo g = grad_geo(s, elem);
    const int64_t Mp = cdiv(s.M, 16) * 16;
    size_t o = 0;
    auto take = [&](size_t n) { size_t r = o; o = align_up(o + n * elem, 256); return r; };
    p.off_gc = take(Mp * Mp);
    p.off_ref = take(2 * s.Q);
    p.off_rowg = take(g.groups > 1 ? (size_t)g.groups * 2 * s.N * s.Q : 0);
    // as many chunks as the region has room for
    const size_t per = (size_t)(s.M * s.Q + g.groups * (s.Q + 1)) * elem;
    const int64_t room = budget > o + 512 ? (int64_t)((budget - o - 512) / per) : 0;
    if (room < 1) return p;  // ok = false
    if (g.chunks > room) {
        const int R = grad_rows(ks_of(s.Q), elem);
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

template <typename T>
hipError_t tiles_psi2_grads(const Shape &s, const TilesGradPlan &p, const T *mu, const T *S, const T *Z,
                            const T *w1, const T *w2, const T *lp1, const T *lp2, const Hyp<T> &h,
                            const T *G1, const T *Gc, T *dmu, T *dS, void *ws, const int *gate,
                            hipStream_t st) {
    const int nb = (int)cdiv(s.M, 16);
    // one group of columns writes dmu and dS themselves
    T *om = p.groups > 1 ? at<T>(ws, p.off_rowg) : dmu;
    T *os = p.groups > 1 ? om + s.N * s.Q : dS;
    const dim3 grid((unsigned)p.groups, (unsigned)p.chunks);
    TimedScope ts(st, "tiles_psi2_grad");
#define GPPS_TILES_GRAD(KS)                                                                       \
    case KS: {                                                                                    \
        const hipError_t e = hipFuncSetAttribute((const void *)tiles_grad_kernel<T, KS>,          \
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,      \
                                                 (int)p.lds);                                     \
        if (e != hipSuccess) return e;                                                            \
        tiles_grad_kernel<T, KS><<<grid, p.nw * 64, p.lds, st>>>(                                 \
            gate, s.N, (int)s.M, (int)s.Q, nb, p.wrows, p.nwin, p.rows, mu, S, Z, w1, w2, lp1,    \
            lp2, h, G1, Gc, at<T>(ws, p.off_ref), om, os, at<T>(ws, p.off_colp),                  \
            at<T>(ws, p.off_rowp));                                                               \
        break;                                                                                    \
    }
    switch (ks_of(s.Q)) {
        GPPS_TILES_GRAD(1) GPPS_TILES_GRAD(2) GPPS_TILES_GRAD(3) GPPS_TILES_GRAD(4)
        GPPS_TILES_GRAD(5) GPPS_TILES_GRAD(6) GPPS_TILES_GRAD(8) GPPS_TILES_GRAD(10)
        GPPS_TILES_GRAD(12) GPPS_TILES_GRAD(16)
        default: return hipErrorInvalidValue;
    }
#undef GPPS_TILES_GRAD
    return hipGetLastError();
}

#define GPPS_TILES_INST(T)                                                                        \
    template hipError_t tiles_psi2<T>(const Shape &, const T *, const T *, const T *, const T *,  \
                                      const T *, const T *, const Hyp<T> &, T *, T *, T *, int,   \
                                      void *, size_t, const int *, hipStream_t);                  \
    template hipError_t tiles_psi2_grads<T>(const Shape &, const TilesGradPlan &, const T *,      \
                                            const T *, const T *, const T *, const T *,           \
                                            const T *, const T *, const Hyp<T> &, const T *,      \
                                            const T *, T *, T *, void *, const int *, hipStream_t);
GPPS_TILES_INST(float)
GPPS_TILES_INST(double)
#undef GPPS_TILES_INST

}  // namespace gpps
