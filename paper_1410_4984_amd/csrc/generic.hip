// Generic path: RBF-ARD psi-statistics and gradients in the element type's own
// arithmetic (float or double).
//
// What is computed (section 2, eq. (4): phi, Phi and Psi become expectations
// under q(x_n) = N(mu_n, diag S_n); Alg. 1 and Alg. 2).  With
//   w1 = 1 / (l^2 + S),  w2 = 1 / (l^2 + 2 S)                          per (n, q)
//   lp1_n = log sf2   - 1/2 sum_q log(1 + S/l^2)
//   lp2_n = 2 log sf2 - 1/2 sum_q log(1 + 2 S/l^2)
// the exact Gaussian integrals give
//   Psi1[n, m]    = exp(lp1_n - 1/2 sum_q (mu - z_m)^2 w1)
//   Psi2_n[m, m'] = exp(lp2_n - sum_q [(z_m - z_m')^2 / (4 l^2) + (mu - zbar)^2 w2])
// with zbar = (z_m + z_m') / 2, and Psi2 = sum_n Psi2_n.
//
// Work split: Psi1 one thread per output.  Psi2 and its gradients go to the 16 x 16 tile
// kernels but at small Q (tiles_stats_wanted, tiles_grads_wanted), where these stay:
//   * Psi2: one thread per unique pair (m <= m'), partial sums per row chunk reduced in a
//     fixed order;
//   * gradients: one thread per inducing input m, the Z table in LDS, per row the sums r
//     and V over the partners m' (symmetric form: each unordered pair evaluated once).
// Fixed-order reduce kernels combine the partials.  No atomics anywhere.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.h"
#include "psi1.h"

namespace gpps {
namespace {

constexpr int kFwdTile = 128;    // rows staged in LDS at a time by the forward pair kernel
constexpr int kPairTile = 16;    // pair tile edge (16 x 16 threads)
constexpr int kBand = 8;         // symmetric pairs kernel: pair offsets k per LDS exchange
constexpr int kSlotBand = 4;     // ... the same with several rows at a time
constexpr int64_t kGridCap = 2048;  // workgroups of the grid-stride kernels

__device__ inline float dexp(float x) { return __expf(x); }
__device__ inline double dexp(double x) { return exp(x); }
__device__ inline float dlog1p(float x) { return log1pf(x); }
__device__ inline double dlog1p(double x) { return log1p(x); }

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Register width (latent dimensions, padded) of the pair kernels for Q <= 4.
inline int64_t pairs_qm(int64_t Q) { return Q <= 1 ? 1 : Q <= 2 ? 2 : 4; }

// The largest workspace before the route word that gpps_psi_stats_noalloc takes.
constexpr size_t kScratchRoom = size_t(GPPS_SCRATCH_BYTES) - 256;

struct Plan {
    bool tstats, tgrads;             // Psi2 / its gradients by the tile kernels
    int64_t tiles_edge;              // pair tiles per edge (Psi2 reduce)
    int64_t pblocks;                 // forward: blocks of 256 unique pairs
    int64_t nc2;                     // row chunks of the Psi2 forward kernel
    int64_t rows2;                   // rows per chunk (forward)
    bool psym;                       // gradients: symmetric form (one workgroup spans all of M)
    bool pslots;                     // ... with R rows at a time (grad_pairs_slots_kernel)
    int prs, psthreads;              // its rows at a time and threads per workgroup
    int pthreads;                    // pairs kernel: threads (inducing inputs) per workgroup
    int64_t pmb, pchunks, prows;     // pairs kernel: m-blocks, row chunks, rows per chunk
    // workspace offsets in bytes; the tile kernels carve the region from off_p2 on
    size_t off_w1, off_w2, off_lp1, off_lp2, off_p2, off_g2s, off_gc, off_colp, off_rowp, off_rowg,
        total;
};

Plan carve(const Shape &s, size_t elem, bool few_rows) {
    Plan p{};
    p.tstats = tiles_stats_wanted(s, elem);
    p.tgrads = tiles_grads_wanted(s, elem);
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t r = o; o = align_up(o + bytes, 256); return r; };
    p.off_w1 = take(elem * s.N * s.Q);
    p.off_w2 = take(elem * s.N * s.Q);
    p.off_lp1 = take(elem * s.N);
    p.off_lp2 = take(elem * s.N);
    p.off_p2 = o;
    if (!p.tstats) {
        p.tiles_edge = cdiv(s.M, kPairTile);
        p.pblocks = cdiv(s.P, 256);
        // 256 rows a chunk, fewer where the chunks are too few for the chip (a chunk's rows
        // are summed one after another: 55 us for 200 rows of Q = 20 in one chunk)
        const int64_t cap2 = std::max<int64_t>(1, 2048 / p.pblocks);
        const int64_t nc2 =
            std::max(cdiv(s.N, 256), few_rows ? std::min(cdiv(s.N, 16), cdiv(256, p.pblocks)) : 0);
        p.nc2 = std::max<int64_t>(1, std::min(nc2, cap2));
        p.rows2 = cdiv(s.N, p.nc2);
        p.nc2 = cdiv(s.N, p.rows2);
        take(elem * p.nc2 * s.P);
    }
    if (!p.tgrads) {
        // one thread per inducing input, the whole Z table (at most 64 KB) in LDS
        const int64_t qm = pairs_qm(s.Q);
        p.pthreads = (int)std::min<int64_t>(256, cdiv(s.M, 64) * 64);
        p.pmb = cdiv(s.M, p.pthreads);
        p.pchunks = std::max<int64_t>(1, std::min<int64_t>(s.N, 2048 / p.pmb));
        p.prows = cdiv(s.N, p.pchunks);
        p.pchunks = cdiv(s.N, p.prows);
        // symmetric form: every pair exchange stays inside one workgroup, and the Z
        // table plus two bands of kBand x M pair values fit in LDS
        p.psym = p.pmb == 1 && (qm + 2 * kBand) * s.M * elem <= 65536;
        p.prs = (int)std::min<int64_t>(8, 512 / s.M);
        p.psthreads = (int)(cdiv(p.prs * s.M, 64) * 64);
        p.pslots = p.psym && p.prs >= 2 &&
                   (s.M * qm + p.prs * 2 * kSlotBand * s.M + p.prs * s.M * 2 * qm) * elem <= 65536;
        if (p.pslots) {
            // chunks a whole number of passes of R rows, about five rounds of two
            // 512-thread workgroups per CU
            p.pchunks = std::max<int64_t>(1, std::min<int64_t>(s.N, 2560));
            p.prows = cdiv(cdiv(s.N, p.pchunks), p.prs) * p.prs;
            p.pchunks = cdiv(s.N, p.prows);
        }
        size_t end = o;
        o = p.off_p2;   // gradients and statistics share the region
        p.off_g2s = take(elem * s.M * s.M);
        p.off_gc = take(elem * (s.M / 2 + 1) * s.M);
        p.off_colp = take(elem * p.pchunks * s.M * s.Q);
        p.off_rowp = take(elem * p.pmb * p.pchunks * (s.Q + 1));
        p.off_rowg = take(elem * (p.pmb > 1 ? p.pmb : 0) * s.N * s.Q * 2);
        o = std::max(o, end);
    }
    // The tile kernels' chunks take what the shape's workspace has in any case (the
    // known-input path's), or what keeps it within GPPS_SCRATCH_BYTES: the
    // allocation-free entry point takes no more.
    const TilesRegion t = tiles_region(s, elem);
    o = std::max(o, p.off_p2 + t.least);
    p.total = o > kScratchRoom
                  ? std::max(o, p.off_p2 + t.want)
                  : std::max(o, std::min(p.off_p2 + t.want,
                                         std::max(kScratchRoom, known_workspace_bytes(s, elem))));
    return p;
}

Plan make_plan(const Shape &s, size_t elem) {
    // the forward's short chunks, unless their partial sums would take the call past
    // the allocation-free entry point's scratch
    const Plan p = carve(s, elem, true);
    return p.total <= kScratchRoom ? p : carve(s, elem, false);
}

template <typename T>
T *at(void *ws, size_t off) { return reinterpret_cast<T *>(static_cast<char *>(ws) + off); }

// ---------------------------------------------------------------- per-row tables
// Workgroups below rblocks: one thread per (row, dimension) for the reciprocals and
// logarithms, then one per row for its sums over q, in the order of q.  One thread
// per row took its 2 Q logarithms one after another: 60 us at N = 100,000, Q = 20
// in fp64 (30 us here), and 15 us of latency in the smallest calls.  The workgroups
// past them lay out the symmetric part of dL/dPsi2 (a launch less per call):
//   kSymPlain  G2s[m][m'] = (G2 + G2^T)/2
//   kSymCirc   Gc[k][m] = G2s[m][(m + k) mod M], k = 0 .. M/2: the symmetric pairs
//              kernel reads the pair (m, m + k) of every thread m as one coalesced row
//   kSymPadded G2s o exp(-sum_q (z_m - z_m')^2 / (4 l^2)), zero-padded to Mp x Mp (the
//              tile kernels; the last Q workgroups then find the centre and the
//              variance of Z in a dimension each, zref [2][Q])
constexpr int kPreElems = 1024;   // (row, dimension) pairs per workgroup
enum SymMode { kSymNone, kSymPlain, kSymCirc, kSymPadded };

template <typename T>
__global__ __launch_bounds__(256) void pre_kernel(const int *__restrict__ gate, int *__restrict__ mark,
                                                  int64_t N, int Q, int rows,
                                                  unsigned rblocks, const T *__restrict__ S, Hyp<T> h,
                                                  T *__restrict__ w1, T *__restrict__ w2,
                                                  T *__restrict__ lp1, T *__restrict__ lp2, int mode,
                                                  int M, int Mp, const T *__restrict__ G2,
                                                  const T *__restrict__ Z, T *__restrict__ G2s,
                                                  unsigned sblocks, T *__restrict__ zref) {
    if (gate && gate[0] == 0) return;
    if (mark && blockIdx.x == 0 && threadIdx.x == 0) mark[0] = 2;
    __shared__ T sl1[kPreElems], sl2[kPreElems];
    if (blockIdx.x >= rblocks + sblocks) {
        const int q = blockIdx.x - rblocks - sblocks;
        auto total = [&](T v) {
            __syncthreads();
            sl1[threadIdx.x] = v;
            __syncthreads();
            for (int w = 128; w >= 1; w >>= 1) {
                if ((int)threadIdx.x < w) sl1[threadIdx.x] += sl1[threadIdx.x + w];
                __syncthreads();
            }
            return sl1[0];
        };
        T a = 0, b = 0;
        for (int m = threadIdx.x; m < M; m += 256) a += Z[(int64_t)m * Q + q];
        const T c = total(a) / T(M);
        for (int m = threadIdx.x; m < M; m += 256) {
            const T d = Z[(int64_t)m * Q + q] - c;
            b += d * d;
        }
        b = total(b) / T(M);
        if (threadIdx.x == 0) {
            zref[q] = c;
            zref[Q + q] = b;
        }
        return;
    }
    if (blockIdx.x >= rblocks) {
        const int64_t i = (int64_t)(blockIdx.x - rblocks) * 256 + threadIdx.x;
        if (mode == kSymCirc) {
            if (i >= (int64_t)(M / 2 + 1) * M) return;
            const int k = (int)(i / M), m = (int)(i - (int64_t)k * M);
            int mp = m + k;
            if (mp >= M) mp -= M;
            G2s[i] = T(0.5) * (G2[(int64_t)m * M + mp] + G2[(int64_t)mp * M + m]);
            return;
        }
        const int W = mode == kSymPadded ? Mp : M;
        if (i >= (int64_t)W * W) return;
        const int m = (int)(i / W), mp = (int)(i - (int64_t)m * W);
        T v = 0;
        if (m < M && mp < M) {
            v = T(0.5) * (G2[(int64_t)m * M + mp] + G2[(int64_t)mp * M + m]);
            if (mode == kSymPadded) {
                T C = 0;
                for (int q = 0; q < Q; ++q) {
                    const T dz = Z[(int64_t)m * Q + q] - Z[(int64_t)mp * Q + q];
                    C -= dz * dz / (T(4) * h.l2[q]);
                }
                v *= dexp(C);
            }
        }
        G2s[i] = v;
        return;
    }
    for (int64_t n0 = (int64_t)blockIdx.x * rows; n0 < N; n0 += (int64_t)rblocks * rows) {
        const int cnt = (int)min<int64_t>(rows, N - n0);
        __syncthreads();
        for (int i = threadIdx.x; i < cnt * Q; i += 256) {
            const T s = S[n0 * Q + i], l2 = h.l2[i % Q];
            w1[n0 * Q + i] = T(1) / (l2 + s);
            w2[n0 * Q + i] = T(1) / (l2 + T(2) * s);
            sl1[i] = dlog1p(s / l2);
            sl2[i] = dlog1p(T(2) * s / l2);
        }
        __syncthreads();
        for (int i = threadIdx.x; i < 2 * cnt; i += 256) {
            const int r = i >> 1;
            const T *sl = (i & 1 ? sl2 : sl1) + r * Q;
            T a = (i & 1 ? T(2) : T(1)) * h.log_sf2;
            for (int q = 0; q < Q; ++q) a -= T(0.5) * sl[q];
            (i & 1 ? lp2 : lp1)[n0 + r] = a;
        }
    }
}

__device__ inline int64_t pair_index(int64_t m, int64_t mp, int64_t M) {
    return m * M - m * (m - 1) / 2 + (mp - m);
}

// Inverse of pair_index: the pair (m, mp), m <= mp, at position t < M (M + 1) / 2
// of the row-major upper triangle.  Row m starts at m (2M - m + 1) / 2; the
// square-root estimate of m is corrected by exact integer tests.
__device__ inline void pair_coords(int64_t t, int64_t M, int &m, int &mp) {
    auto start = [&](int64_t r) { return r * (2 * M - r + 1) / 2; };
    const double b = 2.0 * (double)M + 1.0;
    int64_t r = (int64_t)((b - sqrt(fmax(b * b - 8.0 * (double)t, 0.0))) * 0.5);
    r = r < 0 ? 0 : (r >= M ? M - 1 : r);
    while (r > 0 && start(r) > t) --r;
    while (r + 1 < M && start(r + 1) <= t) ++r;
    m = (int)r;
    mp = (int)(r + (t - start(r)));
}

// ---------------------------------------------------------------- Psi2 partials (Alg. 1, Phi)
// Q <= 4: one thread per unique pair (in the row-major order of the upper triangle, so
// that no lane idles below the diagonal) and row chunk.  The rows' (mu, w2) are
// staged in LDS as pairs.
template <typename T>
struct Two;
template <>
struct Two<float> {
    typedef float2 t;
};
template <>
struct Two<double> {
    typedef double2 t;
};

template <typename T, int QM>
__global__ __launch_bounds__(256) void psi2_partial_kernel(const int *__restrict__ gate,
    int64_t N, int M, int Q, int64_t P, int64_t rows_per_chunk,
    const T *__restrict__ mu, const T *__restrict__ Z, const T *__restrict__ w2,
    const T *__restrict__ lp2, Hyp<T> h, T *__restrict__ partial) {
    if (gate && gate[0] == 0) return;
    using T2 = typename Two<T>::t;
    __shared__ T2 s_mw[kFwdTile][QM];
    __shared__ T s_lp[kFwdTile];
    const int64_t t0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
    // loads from clamped (valid) addresses, masked by a multiplication: a select
    // around each load would let the compiler wait for the loads one at a time
    T zbar[QM], C = 0;
    int m = 0, mp = 0;
    if (t0 < P) pair_coords(t0, M, m, mp);
#pragma unroll
    for (int q = 0; q < QM; ++q) {
        const int qc = min(q, Q - 1);
        const T a = Z[(int64_t)m * Q + qc], b = Z[(int64_t)mp * Q + qc];
        const T on = q < Q ? T(1) : T(0);
        zbar[q] = on * (T(0.5) * (a + b));
        C -= on * ((a - b) * (a - b) / (T(4) * h.l2[qc]));
    }
    const int64_t r0 = (int64_t)blockIdx.y * rows_per_chunk;
    const int64_t r1 = min(N, r0 + rows_per_chunk);
    T acc = 0;
    for (int64_t base = r0; base < r1; base += kFwdTile) {
        const int cnt = (int)min<int64_t>(kFwdTile, r1 - base);
        __syncthreads();
        // zero beyond Q, so that the padded dimensions need no test below; four
        // entries per thread have their loads in flight together
        for (int i0 = threadIdx.x; i0 < cnt * QM; i0 += 4 * blockDim.x) {
            T a[4], b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = min(i0 + u * (int)blockDim.x, cnt * QM - 1);
                const int r = i / QM, q = min(i - r * QM, Q - 1);
                a[u] = mu[(base + r) * Q + q];
                b[u] = w2[(base + r) * Q + q];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + u * (int)blockDim.x;
                const int r = i / QM, q = i - r * QM;
                if (i < cnt * QM) {
                    T2 v;
                    v.x = q < Q ? a[u] : T(0);
                    v.y = q < Q ? b[u] : T(0);
                    s_mw[r][q] = v;
                }
            }
        }
        for (int r = threadIdx.x; r < cnt; r += blockDim.x) s_lp[r] = lp2[base + r];
        __syncthreads();
        // two-level sum: the tile's rows first, then into the chunk total, so
        // that rounding grows with tile + tiles per chunk, not rows per chunk
        T tacc = 0;
#pragma unroll 4
        for (int r = 0; r < cnt; ++r) {
            T e = s_lp[r] + C;
#pragma unroll
            for (int q = 0; q < QM; ++q) {
                const T2 v = s_mw[r][q];
                const T d = v.x - zbar[q];
                e -= d * d * v.y;
            }
            tacc += dexp(e);
        }
        acc += tacc;
    }
    if (t0 < P) partial[(int64_t)blockIdx.y * P + t0] = acc;
}

// Workgroups below edge^2: fixed-order sum of the chunk partials (16 x 16 pairs
// each); both triangles and psi0.  The workgroups past them compute Psi1.
template <typename T>
__global__ __launch_bounds__(256) void psi2_reduce_kernel(
    const int *__restrict__ gate, int64_t N, int M, int Q, int64_t P, int edge, int64_t nchunks,
    const T *__restrict__ partial, Hyp<T> h, T *__restrict__ psi0, T *__restrict__ Psi2, int accumulate,
    const T *__restrict__ mu, const T *__restrict__ Z, const T *__restrict__ w1,
    const T *__restrict__ lp1, T *__restrict__ Psi1) {
    if (gate && gate[0] == 0) return;
    __shared__ Psi1Lds<T> s_p1;
    if (blockIdx.x >= (unsigned)(edge * edge)) {
        psi1_blocks<T>(s_p1, blockIdx.x - edge * edge, gridDim.x - edge * edge, N, M, Q, mu, Z, w1, lp1,
                       Psi1, [](T x) { return dexp(x); });
        return;
    }
    const int bx = blockIdx.x % edge, by = blockIdx.x / edge;
    const int mp = bx * kPairTile + threadIdx.x % kPairTile;
    const int m = by * kPairTile + threadIdx.x / kPairTile;
    if (blockIdx.x == 0 && threadIdx.x == 0)
        psi0[0] = (accumulate ? psi0[0] : T(0)) + T(N) * h.sf2;
    if (m >= M || mp >= M || m > mp) return;
    const int64_t p = pair_index(m, mp, M);
    // chunk order; loads issued 16 at a time so that they overlap
    T s = 0;
    int64_t c = 0;
    for (; c + 16 <= nchunks; c += 16) {
        T v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = partial[(c + j) * P + p];
#pragma unroll
        for (int j = 0; j < 16; ++j) s += v[j];
    }
    for (; c < nchunks; ++c) s += partial[c * P + p];
    T v = (accumulate ? Psi2[(int64_t)m * M + mp] : T(0)) + s;
    Psi2[(int64_t)m * M + mp] = v;
    Psi2[(int64_t)mp * M + m] = v;
}

// ---------------------------------------------------------------- gradients (Alg. 2)
// Psi2 and Psi1 gradients through per-(n, m) sums.  With W_n[m, m'] =
// G2s[m, m'] Psi2_n[m, m'], d = mu_n - z_m, w1 = 1/(l^2 + S_n), w2 = 1/(l^2 + 2 S_n),
//   r_nm = sum_m' W_n[m, m'],  V_nmq = sum_m' W_n[m, m'] d_nm'q,
//   t_nm = dL/dPsi1[n, m] Psi1[n, m],
// every gradient is a sum over (n, m) of (W is symmetric, so the double sum over
// ordered pairs folds onto the m index):
//   dmu_nq += -2 w2 d r - t d w1
//   dS_nq  += w2^2 (d^2 r + d V) - w2 r + t (d^2 w1^2 - w1) / 2
//   dZ_mq  += w2 (d r + V) - (V - d r) / l^2 + t d w1
//   dl_q   += (2 S w2 / l) r + (d^2 r - d V) / l^3 + l w2^2 (d^2 r + d V)
//             + t (S w1 / l + l d^2 w1^2)
//   dsf2   += (2 r + t) / sf2.
// One workgroup per (block of inducing inputs, row chunk), one thread per m, the
// Z table in LDS: dZ_m stays in the thread's registers over the chunk, and per
// row the dmu / dS contributions are summed over the block's m (wave
// butterflies, then the waves in order) into om and os: [m-block][2][N][Q], or dmu and
// dS themselves where one m-block holds all of M.
// Ordered form (SYM = false): thread m evaluates W for every (m, m').
// Symmetric form (SYM = true, the workgroup holds all M): each unordered pair
// is evaluated once.  Thread m takes the pairs (m, m + k mod M) for k = 0 ..
// M/2 (k = M/2 only for m < M/2 when M is even), so every thread has the same
// load; it adds W to its own r and V and leaves it in an LDS band, from which
// thread m + k adds it to its r and V.  The bands hold kBand offsets and are
// double buffered: one barrier per band.
template <typename T, int QM, bool SYM>
__global__ __launch_bounds__(256) void grad_pairs_kernel(const int *__restrict__ gate, 
    int64_t N, int M, int Q, int64_t rows_per_chunk, const T *__restrict__ mu,
    const T *__restrict__ S, const T *__restrict__ Z, const T *__restrict__ w1t,
    const T *__restrict__ w2t, const T *__restrict__ lp1, const T *__restrict__ lp2, Hyp<T> h,
    const T *__restrict__ G1, const T *__restrict__ G2s, const T *__restrict__ Gc,
    T *__restrict__ om, T *__restrict__ os, T *__restrict__ colpart, T *__restrict__ rowpart) {
    if (gate && gate[0] == 0) return;
    extern __shared__ double gp_smem[];
    T *sz = reinterpret_cast<T *>(gp_smem);  // [M][QM], zero beyond Q
    T *band = sz + M * QM;                    // [2][kBand][M] (symmetric form)
    __shared__ T red[2][4][2 * QM];           // per-wave row sums, double buffered by row
    const int tid = threadIdx.x, nthr = blockDim.x, nw = nthr >> 6, wv = tid >> 6;
    const int m = blockIdx.x * nthr + tid;
    const bool valid = m < M;
    for (int i = tid; i < M * QM; i += nthr) {
        const int mm = i / QM, q = i - mm * QM;
        sz[i] = q < Q ? Z[(int64_t)mm * Q + q] : T(0);
    }
    __syncthreads();
    T z[QM], c4[QM], il2[QM], gz[QM], gl[QM];
#pragma unroll
    for (int q = 0; q < QM; ++q) {
        z[q] = valid ? sz[m * QM + q] : T(0);
        c4[q] = q < Q ? T(0.25) / h.l2[q] : T(0);
        il2[q] = q < Q ? T(1) / h.l2[q] : T(0);
        gz[q] = gl[q] = 0;
    }
    T gsf = 0;
    const int K = M / 2;
    const bool even = (M & 1) == 0;
    const int Ku = even ? K - 1 : K;  // offsets taken by every thread
    int band_no = 0;
    const T gdiag = (SYM && valid) ? Gc[m] : T(0);  // G2s[m][m], the same for every row
    const int64_t r0 = (int64_t)blockIdx.y * rows_per_chunk, r1 = min(N, r0 + rows_per_chunk);
    for (int64_t n = r0; n < r1; ++n) {
        T x[QM], a1[QM], a2[QM], sv[QM], d[QM];
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            const bool in = q < Q;
            x[q] = in ? mu[n * Q + q] : T(0);
            a1[q] = in ? w1t[n * Q + q] : T(0);
            a2[q] = in ? w2t[n * Q + q] : T(0);
            sv[q] = in ? S[n * Q + q] : T(0);
            d[q] = x[q] - z[q];
        }
        T r = 0, V[QM];
#pragma unroll
        for (int q = 0; q < QM; ++q) V[q] = 0;
        // W_n[m, m'] = G2s[m, m'] Psi2_n[m, m'] for the partner m' (z row zr).
        // With v = z_m' - z_m and d = mu_n - z_m the exponent
        //   log Psi2 - log prefactor = -sum_q [c4 v^2 + (a2/4)(2 d - v)^2]
        // is a quadratic in v with per-(n, m) coefficients:
        //   e0 + sum_q v (a2 d - (c4 + a2/4) v),  e0 = lp2 - sum_q a2 d^2.
        // Where W is not negligible (exponent above about -30) each of its terms
        // is bounded by a few hundred, so the rounding stays near that of the
        // summed squares.
        T bq[QM], cq[QM], e0 = G2s ? lp2[n] : T(0);
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            bq[q] = a2[q] * d[q];
            cq[q] = c4[q] + T(0.25) * a2[q];
            e0 -= bq[q] * d[q];
        }
        auto pair_w = [&](const T *zr, T g, T e00) {
            T e = e00;
#pragma unroll
            for (int q = 0; q < QM; ++q) {
                const T v = zr[q] - z[q];
                e = fma(v, fma(-cq[q], v, bq[q]), e);
            }
            return g * dexp(e);
        };
        auto add_w = [&](T W, const T *zr) {
            r += W;
#pragma unroll
            for (int q = 0; q < QM; ++q) V[q] += W * (x[q] - zr[q]);
        };
        if (SYM) {
            if (G2s) {  // uniform: every thread reaches the band barriers
                if (valid) add_w(pair_w(sz + m * QM, gdiag, e0), sz + m * QM);
                // offsets every thread takes (1 .. Ku), in bands; then, for even
                // M, the offset M/2 of the first half
                for (int k0 = 1; k0 <= Ku; k0 += kBand, ++band_no) {
                    T *bs = band + (band_no & 1) * (kBand * M);
                    const int k1 = min(Ku, k0 + kBand - 1);
                    if (valid) {
                        int mp = m + k0;
                        if (mp >= M) mp -= M;
                        const T *gk = Gc + (int64_t)k0 * M + m;
#pragma unroll 2
                        for (int k = k0; k <= k1; ++k) {
                            const T W = pair_w(sz + mp * QM, *gk, e0);
                            add_w(W, sz + mp * QM);
                            bs[(k - k0) * M + m] = W;
                            gk += M;
                            mp = mp + 1 == M ? 0 : mp + 1;
                        }
                    }
                    __syncthreads();
                    if (valid) {
                        int sp = m - k0;
                        if (sp < 0) sp += M;
#pragma unroll 4
                        for (int k = k0; k <= k1; ++k) {
                            add_w(bs[(k - k0) * M + sp], sz + sp * QM);
                            sp = sp == 0 ? M - 1 : sp - 1;
                        }
                    }
                }
                if (even && K > 0) {
                    T *bs = band + (band_no & 1) * (kBand * M);
                    ++band_no;
                    if (valid && m < K) {
                        const T W = pair_w(sz + (m + K) * QM, Gc[(int64_t)K * M + m], e0);
                        add_w(W, sz + (m + K) * QM);
                        bs[m] = W;
                    }
                    __syncthreads();
                    if (valid && m >= K) add_w(bs[m - K], sz + (m - K) * QM);
                }
            }
        } else if (G2s && valid) {
            for (int mp = 0; mp < M; ++mp)  // G2s symmetric: G2s[mp][m] is a coalesced row
                add_w(pair_w(sz + mp * QM, G2s[(int64_t)mp * M + m], e0), sz + mp * QM);
        }
        T t = 0;
        if (G1 && valid) {
            T e1 = 0;
#pragma unroll
            for (int q = 0; q < QM; ++q) e1 += d[q] * d[q] * a1[q];
            t = G1[n * M + m] * dexp(lp1[n] - T(0.5) * e1);
        }
        T rv[2 * QM];
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            const T dq = d[q], d2 = dq * dq, dr = dq * r, dV = dq * V[q];
            rv[q] = -T(2) * a2[q] * dr - t * dq * a1[q];
            rv[QM + q] = a2[q] * a2[q] * (d2 * r + dV) - a2[q] * r +
                         T(0.5) * t * (d2 * a1[q] * a1[q] - a1[q]);
            gz[q] += a2[q] * (dr + V[q]) - (V[q] - dr) * il2[q] + t * dq * a1[q];
            if (q < Q) {
                const T l = h.l[q];
                gl[q] += (T(2) * sv[q] * a2[q] / l) * r + (d2 * r - dV) * il2[q] / l +
                         l * a2[q] * a2[q] * (d2 * r + dV) +
                         t * (sv[q] * a1[q] / l + l * d2 * a1[q] * a1[q]);
            }
        }
        gsf += T(2) * r + t;
        // sum of rv over the block's m: butterflies within each wave, then the
        // waves in order (double buffered by row parity: one barrier per row)
        const int b = (int)(n & 1);
#pragma unroll
        for (int k = 0; k < 2 * QM; ++k) {
            T v = rv[k];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
            if ((tid & 63) == 0) red[b][wv][k] = v;
        }
        __syncthreads();
        if (tid < 2 * Q) {
            const int k = tid < Q ? tid : QM + (tid - Q);
            T v = 0;
            for (int w = 0; w < nw; ++w) v += red[b][w][k];
            const int q = tid < Q ? tid : tid - Q;
            (tid < Q ? om : os)[((int64_t)blockIdx.x * 2 * N + n) * Q + q] = v;
        }
    }
    if (valid) {
#pragma unroll
        for (int q = 0; q < QM; ++q)
            if (q < Q) colpart[((int64_t)blockIdx.y * M + m) * Q + q] = gz[q];
    }
    // block sums of dl and dsf2 (fixed order, as above) -> rowpart[block][Q + 1]
    const int64_t blk = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    __syncthreads();
#pragma unroll
    for (int k = 0; k <= QM; ++k) {
        if (k < Q || k == QM) {
            T v = k < QM ? gl[k] : gsf / h.sf2;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
            if ((tid & 63) == 0) red[0][wv][0] = v;
            __syncthreads();
            if (tid == 0) {
                T s = 0;
                for (int w = 0; w < nw; ++w) s += red[0][w][0];
                rowpart[blk * (Q + 1) + (k < QM ? k : Q)] = s;
            }
            __syncthreads();
        }
    }
}

// The band form with R = min(8, 512 / M) rows at a time, so that a workgroup
// of R M threads (rounded up to whole waves) leaves few lanes idle when M is
// not a multiple of 64.  Thread (slot, m) = (tid / M, tid % M) works on row
// r0 + it R + slot of pass it; each slot exchanges W through its own double
// buffered band of kSlotBand offsets.  Per row the dmu / dS terms are summed
// over m through LDS (32 lanes per output, each adding m = u, u + 32, ... in
// order, then a fixed butterfly); dZ_m adds the slots in order at the end.

template <typename T, int QM>
__global__ __launch_bounds__(512) void grad_pairs_slots_kernel(const int *__restrict__ gate, 
    int64_t N, int M, int Q, int R, int64_t rows_per_chunk, const T *__restrict__ mu,
    const T *__restrict__ S, const T *__restrict__ Z, const T *__restrict__ w1t,
    const T *__restrict__ w2t, const T *__restrict__ lp1, const T *__restrict__ lp2, Hyp<T> h,
    const T *__restrict__ G1, const T *__restrict__ G2s, const T *__restrict__ Gc,
    T *__restrict__ om, T *__restrict__ os, T *__restrict__ colpart, T *__restrict__ rowpart) {
    if (gate && gate[0] == 0) return;
    extern __shared__ double gs_smem[];
    T *sz = reinterpret_cast<T *>(gs_smem);        // [M][QM], zero beyond Q
    T *band = sz + M * QM;                          // [R][2][kSlotBand][M]
    T *rvs = band + (size_t)R * 2 * kSlotBand * M;  // [R M][2 QM]: row terms, then dZ by slot
    __shared__ T redw[8];
    const int tid = threadIdx.x, nthr = blockDim.x, nw = nthr >> 6, wv = tid >> 6;
    const int slot = tid / M, m = tid - slot * M;
    const bool valid = slot < R;
    for (int i = tid; i < M * QM; i += nthr) {
        const int mm = i / QM, q = i - mm * QM;
        sz[i] = q < Q ? Z[(int64_t)mm * Q + q] : T(0);
    }
    __syncthreads();
    T z[QM], c4[QM], il2[QM], gz[QM], gl[QM];
#pragma unroll
    for (int q = 0; q < QM; ++q) {
        z[q] = valid ? sz[m * QM + q] : T(0);
        c4[q] = q < Q ? T(0.25) / h.l2[q] : T(0);
        il2[q] = q < Q ? T(1) / h.l2[q] : T(0);
        gz[q] = gl[q] = 0;
    }
    T gsf = 0;
    const int K = M / 2;
    const bool even = (M & 1) == 0;
    const int Ku = even ? K - 1 : K;  // offsets taken by every thread
    int band_no = 0;
    const T gdiag = valid ? Gc[m] : T(0);
    const int64_t r0 = (int64_t)blockIdx.y * rows_per_chunk, r1 = min(N, r0 + rows_per_chunk);
    const int64_t iters = (r1 - r0 + R - 1) / R;
    for (int64_t it = 0; it < iters; ++it) {
        const int64_t n = r0 + it * R + slot;
        const bool rin = valid && n < r1;
        T x[QM], a1[QM], a2[QM], sv[QM], d[QM];
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            const bool in = rin && q < Q;
            x[q] = in ? mu[n * Q + q] : T(0);
            a1[q] = in ? w1t[n * Q + q] : T(0);
            a2[q] = in ? w2t[n * Q + q] : T(0);
            sv[q] = in ? S[n * Q + q] : T(0);
            d[q] = x[q] - z[q];
        }
        T r = 0, V[QM];
#pragma unroll
        for (int q = 0; q < QM; ++q) V[q] = 0;
        // the exponent as a quadratic in v = z_m' - z_m (as in grad_pairs_kernel)
        T bq[QM], cq[QM], e0 = (G2s && rin) ? lp2[n] : T(0);
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            bq[q] = a2[q] * d[q];
            cq[q] = c4[q] + T(0.25) * a2[q];
            e0 -= bq[q] * d[q];
        }
        auto pair_w = [&](const T *zr, T g) {
            T e = e0;
#pragma unroll
            for (int q = 0; q < QM; ++q) {
                const T v = zr[q] - z[q];
                e = fma(v, fma(-cq[q], v, bq[q]), e);
            }
            return g * dexp(e);
        };
        auto add_w = [&](T W, const T *zr) {
            r += W;
#pragma unroll
            for (int q = 0; q < QM; ++q) V[q] += W * (x[q] - zr[q]);
        };
        if (G2s) {  // uniform: every thread reaches the band barriers
            if (rin) add_w(pair_w(sz + m * QM, gdiag), sz + m * QM);
            for (int k0 = 1; k0 <= Ku; k0 += kSlotBand, ++band_no) {
                T *bs = band + ((size_t)slot * 2 + (band_no & 1)) * (kSlotBand * M);
                const int k1 = min(Ku, k0 + kSlotBand - 1);
                if (rin) {
                    int mp = m + k0;
                    if (mp >= M) mp -= M;
                    const T *gk = Gc + (int64_t)k0 * M + m;
#pragma unroll 2
                    for (int k = k0; k <= k1; ++k) {
                        const T W = pair_w(sz + mp * QM, *gk);
                        add_w(W, sz + mp * QM);
                        bs[(k - k0) * M + m] = W;
                        gk += M;
                        mp = mp + 1 == M ? 0 : mp + 1;
                    }
                }
                __syncthreads();
                if (rin) {
                    int sp = m - k0;
                    if (sp < 0) sp += M;
#pragma unroll 4
                    for (int k = k0; k <= k1; ++k) {
                        add_w(bs[(k - k0) * M + sp], sz + sp * QM);
                        sp = sp == 0 ? M - 1 : sp - 1;
                    }
                }
            }
            if (even && K > 0) {
                T *bs = band + ((size_t)slot * 2 + (band_no & 1)) * (kSlotBand * M);
                ++band_no;
                if (rin && m < K) {
                    const T W = pair_w(sz + (m + K) * QM, Gc[(int64_t)K * M + m]);
                    add_w(W, sz + (m + K) * QM);
                    bs[m] = W;
                }
                __syncthreads();
                if (rin && m >= K) add_w(bs[m - K], sz + (m - K) * QM);
            }
        }
        T rv[2 * QM];
#pragma unroll
        for (int k = 0; k < 2 * QM; ++k) rv[k] = 0;
        if (rin) {
            T t = 0;
            if (G1) {
                T e1 = 0;
#pragma unroll
                for (int q = 0; q < QM; ++q) e1 += d[q] * d[q] * a1[q];
                t = G1[n * M + m] * dexp(lp1[n] - T(0.5) * e1);
            }
#pragma unroll
            for (int q = 0; q < QM; ++q) {
                const T dq = d[q], d2 = dq * dq, dr = dq * r, dV = dq * V[q];
                rv[q] = -T(2) * a2[q] * dr - t * dq * a1[q];
                rv[QM + q] = a2[q] * a2[q] * (d2 * r + dV) - a2[q] * r +
                             T(0.5) * t * (d2 * a1[q] * a1[q] - a1[q]);
                gz[q] += a2[q] * (dr + V[q]) - (V[q] - dr) * il2[q] + t * dq * a1[q];
                if (q < Q) {
                    const T l = h.l[q];
                    gl[q] += (T(2) * sv[q] * a2[q] / l) * r + (d2 * r - dV) * il2[q] / l +
                             l * a2[q] * a2[q] * (d2 * r + dV) +
                             t * (sv[q] * a1[q] / l + l * d2 * a1[q] * a1[q]);
                }
            }
            gsf += T(2) * r + t;
        }
        if (valid) {
#pragma unroll
            for (int k = 0; k < 2 * QM; ++k) rvs[(size_t)tid * 2 * QM + k] = rv[k];
        }
        __syncthreads();
        {
            const int g = tid >> 5, u = tid & 31, outs = R * 2 * Q;
            for (int o = g; o < outs; o += nthr >> 5) {
                const int sl = o / (2 * Q), j = o - sl * 2 * Q;
                const int kk = j < Q ? j : QM + (j - Q);
                T v = 0;
                for (int mm = u; mm < M; mm += 32) v += rvs[((size_t)sl * M + mm) * 2 * QM + kk];
#pragma unroll
                for (int off = 16; off >= 1; off >>= 1) v += __shfl_xor(v, off);
                const int64_t nn = r0 + it * R + sl;
                if (u == 0 && nn < r1) {
                    (j < Q ? om : os)[nn * Q + (j < Q ? j : j - Q)] = v;
                }
            }
        }
        __syncthreads();  // rvs is written again in the next pass
    }
    // dZ_m: the slots in order -> colpart[chunk][m][q]
    if (valid) {
#pragma unroll
        for (int q = 0; q < QM; ++q) rvs[((size_t)slot * M + m) * QM + q] = gz[q];
    }
    __syncthreads();
    if (tid < M) {
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            if (q < Q) {
                T v = 0;
                for (int sl = 0; sl < R; ++sl) v += rvs[((size_t)sl * M + tid) * QM + q];
                colpart[((int64_t)blockIdx.y * M + tid) * Q + q] = v;
            }
        }
    }
    // block sums of dl and dsf2 (wave butterflies, then the waves in order) ->
    // rowpart[chunk][Q + 1]
    const int64_t blk = blockIdx.y;
#pragma unroll
    for (int k = 0; k <= QM; ++k) {
        if (k < Q || k == QM) {
            T v = k < QM ? gl[k] : gsf / h.sf2;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
            __syncthreads();
            if ((tid & 63) == 0) redw[wv] = v;
            __syncthreads();
            if (tid == 0) {
                T s2 = 0;
                for (int w = 0; w < nw; ++w) s2 += redw[w];
                rowpart[blk * (Q + 1) + (k < QM ? k : Q)] = s2;
            }
        }
    }
}

// Fixed-order reductions of the gradient partials, one launch.  Workgroups below
// rb: dmu, dS, the nblk partials [nblk][2][N][Q] in block order (none where the
// kernel before wrote them itself).  Then zb workgroups for dZ: with `wide` 32
// entries each, 8 groups of 32 threads taking partials g, g + 8, ... (coalesced) and
// the 8 group sums in order; else one entry at a time, thread t taking partials t,
// t + 256, ... and a fixed tree (few entries of many partials).  Then one per dl_q
// and one for dsf2, by the tree.
template <typename T>
__global__ __launch_bounds__(256) void grad_finish_kernel(
    const int *__restrict__ gate, int64_t N, int M, int Q, unsigned rb, int nblk,
    const T *__restrict__ rowg, T *__restrict__ dmu, T *__restrict__ dS, unsigned zb, int wide,
    int64_t ncol, int64_t nrow, const T *__restrict__ colpart, const T *__restrict__ rowpart,
    T dL_dpsi0, T *__restrict__ dZ, T *__restrict__ dsf2, T *__restrict__ dl, int accumulate) {
    if (gate && gate[0] == 0) return;
    __shared__ T red[256];
    const int t = threadIdx.x;
    if (blockIdx.x < rb) {
        const int64_t NQ = N * Q;
        for (int64_t i = (int64_t)blockIdx.x * 256 + t; i < NQ; i += (int64_t)rb * 256) {
            T a = 0, b = 0;
            for (int r = 0; r < nblk; ++r) {
                a += rowg[(int64_t)(2 * r) * NQ + i];
                b += rowg[(int64_t)(2 * r + 1) * NQ + i];
            }
            dmu[i] = a;
            dS[i] = b;
        }
        return;
    }
    const int64_t MQ = (int64_t)M * Q;
    auto tree = [&](T s) {
        __syncthreads();
        red[t] = s;
        __syncthreads();
        for (int w = 128; w >= 1; w >>= 1) {
            if (t < w) red[t] += red[t + w];
            __syncthreads();
        }
        return red[0];
    };
    const unsigned b = blockIdx.x - rb;
    if (b < zb) {
        if (wide) {
            const int o = t & 31, g = t >> 5;
            for (int64_t i0 = (int64_t)b * 32; i0 < MQ; i0 += (int64_t)zb * 32) {
                const int64_t i = min(i0 + o, MQ - 1);
                T s = 0;
#pragma unroll 8
                for (int64_t c = g; c < ncol; c += 8) s += colpart[c * MQ + i];
                __syncthreads();
                red[t] = s;
                __syncthreads();
                if (g == 0 && i0 + o < MQ) {
                    T v = 0;
                    for (int k = 0; k < 8; ++k) v += red[k * 32 + o];
                    dZ[i] = (accumulate ? dZ[i] : T(0)) + v;
                }
            }
            return;
        }
        for (int64_t i = b; i < MQ; i += zb) {
            T s = 0;
            for (int64_t c = t; c < ncol; c += 256) s += colpart[c * MQ + i];
            s = tree(s);
            if (t == 0) dZ[i] = (accumulate ? dZ[i] : T(0)) + s;
        }
        return;
    }
    const int k = (int)(b - zb);  // k < Q: dl_k; k == Q: dsf2
    T s = 0;
    for (int64_t c = t; c < nrow; c += 256) s += rowpart[c * (Q + 1) + k];
    s = tree(s);
    if (t != 0) return;
    if (k < Q) {
        dl[k] = (accumulate ? dl[k] : T(0)) + s;
    } else {
        s += dL_dpsi0 * T(N);
        dsf2[0] = (accumulate ? dsf2[0] : T(0)) + s;
    }
}

// The per-row tables, and the symmetric part of dL/dPsi2 as `mode` asks.
template <typename T>
void pre(const Shape &s, const Plan &p, const T *S, const Hyp<T> &h, void *ws, const int *gate,
         int *mark, hipStream_t st, int mode = kSymNone, const T *G2 = nullptr, const T *Z = nullptr,
         T *G2s = nullptr, T *zref = nullptr) {
    // few rows a workgroup where there are few: at least a workgroup per CU
    const int64_t rows = std::max<int64_t>(1, std::min(kPreElems / s.Q, cdiv(s.N, 256)));
    const int64_t Mp = cdiv(s.M, 16) * 16;
    const int64_t n = mode == kSymNone ? 0
                      : mode == kSymCirc ? (s.M / 2 + 1) * s.M
                      : mode == kSymPadded ? Mp * Mp : s.M * s.M;
    TimedScope ts(st, "generic_pre");
    const int64_t sb = cdiv(n, 256), zb = zref ? s.Q : 0;
    const int64_t rb = std::min(cdiv(s.N, rows), kMaxBlocks - sb - zb);   // more row blocks: in turn
    pre_kernel<T><<<(unsigned)(rb + sb + zb), 256, 0, st>>>(
        gate, mark, s.N, (int)s.Q, (int)rows, (unsigned)rb, S, h, at<T>(ws, p.off_w1), at<T>(ws, p.off_w2),
        at<T>(ws, p.off_lp1), at<T>(ws, p.off_lp2), mode, (int)s.M, (int)Mp, G2, Z, G2s,
        (unsigned)sb, zref);
}

// nblk > 1: dmu and dS from rowg's partials; else the caller's kernel wrote them.
template <typename T>
void finish(const Shape &s, int64_t nblk, const T *rowg, T *dmu, T *dS, int64_t ncol, int64_t nrow,
            const T *colpart, const T *rowpart, T dL_dpsi0, T *dZ, T *dsf2, T *dl, int accumulate,
            const int *gate, hipStream_t st) {
    const int64_t rb = nblk > 1 ? std::min<int64_t>(cdiv(s.N * s.Q, 256), kGridCap) : 0;
    // 32 entries a workgroup once that leaves four workgroups per CU (the tree reads
    // one value per partial and lane group: 82 us against 20 at 5,120 entries of 1,024)
    const int wide = s.M * s.Q >= 2048 || ncol <= 32;
    const int64_t zb = std::min<int64_t>(wide ? cdiv(s.M * s.Q, 32) : s.M * s.Q, kGridCap);
    TimedScope ts(st, "generic_grad_finish");
    grad_finish_kernel<T><<<(unsigned)(rb + zb + s.Q + 1), 256, 0, st>>>(
        gate, s.N, (int)s.M, (int)s.Q, (unsigned)rb, (int)nblk, rowg, dmu, dS, (unsigned)zb, wide, ncol,
        nrow, colpart, rowpart, dL_dpsi0, dZ, dsf2, dl, accumulate);
}

}  // namespace

size_t generic_workspace_bytes(const Shape &s, size_t elem) { return make_plan(s, elem).total; }

template <typename T>
hipError_t generic_psi_stats(const Shape &s, const T *mu, const T *S, const T *Z,
                             const Hyp<T> &h, T *psi0, T *Psi1, T *Psi2, int accumulate,
                             void *ws, const int *gate, int *mark, hipStream_t st) {
    const Plan p = make_plan(s, sizeof(T));
    pre<T>(s, p, S, h, ws, gate, mark, st);
    const T *w1 = at<T>(ws, p.off_w1), *w2 = at<T>(ws, p.off_w2);
    const T *lp1 = at<T>(ws, p.off_lp1), *lp2 = at<T>(ws, p.off_lp2);
    if (p.tstats)
        return tiles_psi2<T>(s, mu, Z, w1, w2, lp1, lp2, h, psi0, Psi1, Psi2, accumulate,
                             at<char>(ws, p.off_p2),
                             std::max(p.total, known_workspace_bytes(s, sizeof(T))) - p.off_p2, gate, st);
    T *partial = at<T>(ws, p.off_p2);
    {
        const dim3 grid((unsigned)p.pblocks, (unsigned)p.nc2);
        TimedScope ts(st, "generic_psi2_partial");
#define GPPS_FWD(QMV)                                                                              \
    psi2_partial_kernel<T, QMV><<<grid, 256, 0, st>>>(gate, s.N, (int)s.M, (int)s.Q, s.P, p.rows2, \
                                                      mu, Z, w2, lp2, h, partial)
        switch (pairs_qm(s.Q)) {
            case 1: GPPS_FWD(1); break;
            case 2: GPPS_FWD(2); break;
            default: GPPS_FWD(4); break;
        }
#undef GPPS_FWD
    }
    const int64_t tiles = p.tiles_edge * p.tiles_edge;
    TimedScope ts(st, "generic_psi2_reduce_psi1");
    psi2_reduce_kernel<T><<<(unsigned)(tiles + psi1_grid(s.N, s.M, Psi1, kGridCap)), 256, 0, st>>>(
        gate, s.N, (int)s.M, (int)s.Q, s.P, (int)p.tiles_edge, p.nc2, partial, h, psi0, Psi2, accumulate,
        mu, Z, w1, lp1, Psi1);
    return hipGetLastError();
}

template <typename T>
hipError_t generic_psi_grads(const Shape &s, const T *mu, const T *S, const T *Z,
                             const Hyp<T> &h, T dL_dpsi0, const T *G1, const T *G2, T *dmu,
                             T *dS, T *dZ, T *dsf2, T *dl, int accumulate, void *ws,
                             const int *gate, int *mark, hipStream_t st) {
    const Plan p = make_plan(s, sizeof(T));
    const T *w1 = at<T>(ws, p.off_w1), *w2 = at<T>(ws, p.off_w2);
    const T *lp1 = at<T>(ws, p.off_lp1), *lp2 = at<T>(ws, p.off_lp2);
    if (p.tgrads) {
        const TilesGradPlan f = tiles_grad_plan(s, p.total - p.off_p2, sizeof(T));
        if (!f.ok) return hipErrorInvalidValue;   // no shape: the region holds at least one chunk
        char *region = at<char>(ws, p.off_p2);
        T *Gc = G2 ? at<T>(region, f.off_gc) : nullptr;
        T *zref = G2 ? at<T>(region, f.off_ref) : nullptr;
        pre<T>(s, p, S, h, ws, gate, mark, st, G2 ? kSymPadded : kSymNone, G2, Z, Gc, zref);
        const hipError_t e = tiles_psi2_grads<T>(s, f, mu, S, Z, w1, w2, lp1, lp2, h, G1, Gc, dmu, dS,
                                                 region, gate, st);
        if (e != hipSuccess) return e;
        finish<T>(s, f.groups, at<T>(region, f.off_rowg), dmu, dS, f.chunks, f.chunks * f.groups,
                  at<T>(region, f.off_colp), at<T>(region, f.off_rowp), dL_dpsi0, dZ, dsf2, dl,
                  accumulate, gate, st);
        return hipGetLastError();
    }
    T *colpart = at<T>(ws, p.off_colp), *rowpart = at<T>(ws, p.off_rowp);
    T *rowg = at<T>(ws, p.off_rowg);
    const bool sym = p.psym && G2;
    T *G2s = G2 ? at<T>(ws, sym ? p.off_gc : p.off_g2s) : nullptr;
    pre<T>(s, p, S, h, ws, gate, mark, st, !G2 ? kSymNone : sym ? kSymCirc : kSymPlain, G2, Z, G2s);
    // one block of columns writes dmu and dS themselves
    T *om = p.pmb > 1 ? rowg : dmu, *os = p.pmb > 1 ? rowg + s.N * s.Q : dS;
    const size_t lds = sizeof(T) * s.M * (pairs_qm(s.Q) + (sym ? 2 * kBand : 0));
    const size_t lds_slots =
        sizeof(T) * s.M * (pairs_qm(s.Q) + p.prs * 2 * kSlotBand + p.prs * 2 * pairs_qm(s.Q));
    dim3 grid((unsigned)p.pmb, (unsigned)p.pchunks);
    {
        TimedScope ts(st, "generic_grad_pairs");
#define GPPS_PAIRS(QMV)                                                                            \
    do {                                                                                           \
        if (sym && p.pslots)                                                                       \
            grad_pairs_slots_kernel<T, QMV><<<grid, p.psthreads, lds_slots, st>>>(gate,            \
                s.N, (int)s.M, (int)s.Q, p.prs, p.prows, mu, S, Z, w1, w2, lp1, lp2, h, G1, G2s,   \
                G2s, om, os, colpart, rowpart);                                                    \
        else if (sym)                                                                              \
            grad_pairs_kernel<T, QMV, true><<<grid, p.pthreads, lds, st>>>(gate,                   \
                s.N, (int)s.M, (int)s.Q, p.prows, mu, S, Z, w1, w2, lp1, lp2, h, G1, G2s, G2s,     \
                om, os, colpart, rowpart);                                                         \
        else                                                                                       \
            grad_pairs_kernel<T, QMV, false><<<grid, p.pthreads, lds, st>>>(gate,                  \
                s.N, (int)s.M, (int)s.Q, p.prows, mu, S, Z, w1, w2, lp1, lp2, h, G1, G2s, nullptr, \
                om, os, colpart, rowpart);                                                         \
    } while (0)
        switch (pairs_qm(s.Q)) {
            case 1: GPPS_PAIRS(1); break;
            case 2: GPPS_PAIRS(2); break;
            default: GPPS_PAIRS(4); break;
        }
#undef GPPS_PAIRS
    }
    finish<T>(s, p.pmb, rowg, dmu, dS, p.pchunks, p.pmb * p.pchunks, colpart, rowpart, dL_dpsi0, dZ,
              dsf2, dl, accumulate, gate, st);
    return hipGetLastError();
}

template hipError_t generic_psi_stats<float>(const Shape &, const float *, const float *,
                                             const float *, const Hyp<float> &, float *,
                                             float *, float *, int, void *, const int *,
                                             int *, hipStream_t);
template hipError_t generic_psi_stats<double>(const Shape &, const double *, const double *,
                                              const double *, const Hyp<double> &, double *,
                                              double *, double *, int, void *, const int *,
                                              int *, hipStream_t);
template hipError_t generic_psi_grads<float>(const Shape &, const float *, const float *,
                                             const float *, const Hyp<float> &, float,
                                             const float *, const float *, float *, float *,
                                             float *, float *, float *, int, void *,
                                             const int *, int *, hipStream_t);
template hipError_t generic_psi_grads<double>(const Shape &, const double *, const double *,
                                              const double *, const Hyp<double> &, double,
                                              const double *, const double *, double *,
                                              double *, double *, double *, double *, int,
                                              void *, const int *, int *, hipStream_t);

}  // namespace gpps
