// hmm.hip -- discrete-state hidden Markov model: the parallel filter and
// smoother of Sections II-III with a finite state space (integrals become sums
// over the states; the concluding section of the paper notes the framework
// holds there).
//
// Model: x_0 ~ p0, p(x_k = j | x_{k-1} = i) = Pi[i][j], p(y_k | x_k = j) =
// exp(L[k-1][j]) (the caller's emission log-likelihoods).
//
// Filtering (Theorem 1, Definition 1).  The element of step k is the pair
// f_k[z][x] = p(x_k = x | y_k, x_{k-1} = z), g_k[z] = p(y_k | x_{k-1} = z).
// Written as one matrix Psi_k = diag(g_k) f_k, Psi_k[z][x] = Pi[z][x]
// exp(L[k-1][x]) (step 1: p0^T Pi diag(exp L[0]) in every row), Definition 1's
// operator is exactly the matrix product: (Psi_i Psi_j)[z][x] =
// g_i[z] (sum_y f_i[z][y] g_j[y]) f_ij[z][x] = g_ij[z] f_ij[z][x].  A matrix is
// stored row-normalised with a log-scale per row, (A, c): Psi = diag(e^c) A,
// rows of A summing to one (A = f, c = log g).  A row whose weight is zero
// (the data are impossible from that state) is kept as zeros with c = -inf.
// The prefix from step 1 has identical rows: the filtered marginal
// p(x_k | y_1:k) and c = log p(y_1:k).
//
// Smoothing (Theorem 2, Definition 2).  The element of step k < T is
// a_k(x | z) = p(x_k = x | y_1:k, x_{k+1} = z) = alpha_k[x] Pi[x][z] / pred_{k+1}[z]
// with pred_{k+1} = alpha_k^T Pi, and a_T(x | z) = alpha_T[x].  As matrices
// E[z][x] = a(x | z), the operator is E(a_i (x) a_j) = E(a_j) E(a_i); a
// suffix a_k (x) ... (x) a_e is V = E_e ... E_k, built from the right end of a
// block as V <- V diag(1/pred_{k+1}) Pi^T diag(alpha_k).  A state z that the
// filter cannot reach (pred_{k+1}[z] = 0) has no defined row; its column of
// diag(1/pred) is taken as zero (such a row never carries smoothing weight).
//
// Scan: the time axis is cut into blocks of l steps (Section III-C's block
// elements).  Rows of a block's running product evolve independently
// (row z of V Pi only reads row z of V), so wave w of a block's workgroup owns
// rows 16 w .. 16 w + 15 and runs its products on the matrix cores
// (v_mfma_f64_16x16x4f64) with no synchronisation between waves:
//   k_hmm_filter_reduce / k_hmm_smoother_reduce  one workgroup per block:
//       the block element (filter: left to right; smoother: right to left);
//   k_hmm_scan_level   one Hillis-Steele level over the block elements
//       (ceil(log2 nblk) launches, ping-pong buffers), full matrices;
//   k_hmm_filter_down / k_hmm_smoother_down  one wave per block: the
//       incoming prefix (suffix) of a block is a single row, so the block's
//       steps are re-run as the vector recursion alpha_k ∝ (alpha_{k-1}^T Pi)
//       ∘ exp(L[k-1]) (resp. gamma_k = alpha_k ∘ Pi (gamma_{k+1} / pred_{k+1})),
//       exactly Definitions 1 and 2 with a rank-one left (right) operand.
// Long sequences of chains that forget their start do without the block
// elements: see "Overlapped blocks" below.
// States are padded to KP = 16 ceil(K / 16) with zero rows and columns.
// Everything is FP64.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "pks_internal.h"

namespace pks {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

struct HmmArgs {
    int K;                 // states
    int64_t T;             // steps
    int64_t l;             // steps per block
    int64_t nblk;          // blocks
    const double* Pi;      // [K][K]
    const double* p0;      // [K]
    const double* L;       // [T][K] log-likelihoods
    double* alpha;         // [T][K]
    double* logp;          // [T] log p(y_1:k) or nullptr
    double* gamma;         // [T][K]
    double* aggA;          // [nblk][KP][KP] block elements (filter: A; smoother: V)
    double* aggC;          // [nblk][KP] row log-scales (filter)
    double* aggA2;         // ping-pong partner
    double* aggC2;
    const int* skip;       // GATED kernels return at once when *skip is set: the overlapped blocks have done the work
};

__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// sum over the 16 lanes that share lane / 16 (one row of a 16 x 16 tile)
__device__ __forceinline__ double sum16(double v) {
    v += __shfl_xor(v, 1, 16);
    v += __shfl_xor(v, 2, 16);
    v += __shfl_xor(v, 4, 16);
    v += __shfl_xor(v, 8, 16);
    return v;
}
__device__ __forceinline__ double max64(double v) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) v = fmax(v, __shfl_xor(v, m, 64));
    return v;
}
__device__ __forceinline__ double sum64(double v) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// exp(L[k][x] - M_k) for the lane's state x = lane (0 for padded states) and
// M_k = max_x L[k][x]
__device__ __forceinline__ double scaled_lik(const double* __restrict__ Lk, int K, int lane, double& M) {
    const double v = lane < K ? Lk[lane] : -HUGE_VAL;
    M = max64(v);
    return lane < K ? exp(v - M) : 0.0;
}

// ---------------------------------------------------------------------------
// Strip products on the matrix cores.  A 16 x KP strip X (rows of the wave)
// times a KP x KP matrix Y: lane l supplies X(l % 16, 4 s + l / 16) and
// Y(4 s + l / 16, 16 t + l % 16) and receives D(4 v + l / 16, 16 t + l % 16)
// in register v of tile t.  X comes from the wave's LDS stage (row stride KP
// + 1 doubles), Y from registers (Yf[s][t]).
// ---------------------------------------------------------------------------
template <int KP>
__device__ __forceinline__ void strip_times(const double* __restrict__ Xs, const double (&Yf)[KP / 4][KP / 16],
                                            f64x4 (&D)[KP / 16], int li, int lk) {
    constexpr int NT = KP / 16, NS = KP / 4;
#pragma unroll
    for (int t = 0; t < NT; ++t) D[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const double xa = Xs[li * (KP + 1) + 4 * s + lk];
#pragma unroll
        for (int t = 0; t < NT; ++t) D[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa, Yf[s][t], D[t], 0, 0, 0);
    }
}

// write the strip held in D layout into the stage (rows 4 v + lk, columns 16 t + li)
template <int KP>
__device__ __forceinline__ void stage_strip(double* __restrict__ Xs, const f64x4 (&D)[KP / 16], int li, int lk) {
#pragma unroll
    for (int t = 0; t < KP / 16; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) Xs[(4 * v + lk) * (KP + 1) + 16 * t + li] = D[t][v];
}

// Y fragments of Pi (trans = false) or Pi^T (trans = true), zero outside K x K
template <int KP>
__device__ __forceinline__ void load_pi_frags(const double* __restrict__ Pi, int K, bool trans,
                                              double (&Yf)[KP / 4][KP / 16], int li, int lk) {
#pragma unroll
    for (int s = 0; s < KP / 4; ++s)
#pragma unroll
        for (int t = 0; t < KP / 16; ++t) {
            const int r = 4 * s + lk, c = 16 * t + li;
            const int i = trans ? c : r, j = trans ? r : c;
            Yf[s][t] = (r < K && c < K) ? Pi[i * K + j] : 0.0;
        }
}

// ---------------------------------------------------------------------------
// Filter reduce: the block element a_s (x) ... (x) a_e, left to right, starting
// from the identity (A = I, c = 0).  One step: A <- A Pi diag(exp(L_k - M_k)),
// rows renormalised, c += M_k + log(row sum); at the sequence's first step the
// rows of A are first replaced by p0 (a_1 does not depend on x_0).
// ---------------------------------------------------------------------------
template <int KP, bool GATED>
__global__ __launch_bounds__(KP / 16 * 64) void k_hmm_filter_reduce(HmmArgs a) {
    if (GATED && *a.skip != 0) return;
    constexpr int NT = KP / 16;
    __shared__ double stage[NT][16 * (KP + 1)];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
    const int64_t s = (int64_t)blockIdx.x * a.l;
    const int64_t e = min(s + a.l, a.T);
    const int K = a.K;
    double* Xs = stage[w];
    double Yf[KP / 4][NT];
    load_pi_frags<KP>(a.Pi, K, false, Yf, li, lk);
    f64x4 D[NT];
    double c[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        c[v] = 0.0;
#pragma unroll
        for (int t = 0; t < NT; ++t) D[t][v] = (16 * w + 4 * v + lk == 16 * t + li) ? 1.0 : 0.0;
    }
    for (int64_t k = s; k < e; ++k) {
        if (k == 0) {
            const double* p0 = a.p0;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const double pv = (16 * t + li < K) ? p0[16 * t + li] : 0.0;
#pragma unroll
                for (int v = 0; v < 4; ++v) D[t][v] = (16 * w + 4 * v + lk < K) ? pv : 0.0;
            }
        }
        stage_strip<KP>(Xs, D, li, lk);
        wave_sync_lds();
        strip_times<KP>(Xs, Yf, D, li, lk);
        double M;
        const double lh = scaled_lik(a.L + k * K, K, lane, M);
        double rs[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const double lt = __shfl(lh, 16 * t + li, 64);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                D[t][v] *= lt;
                rs[v] += D[t][v];
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double r = sum16(rs[v]);
            const double inv = r > 0.0 ? 1.0 / r : 0.0;
#pragma unroll
            for (int t = 0; t < NT; ++t) D[t][v] *= inv;
            c[v] += M + log(r);
        }
        wave_sync_lds();                     // the stage is rewritten next step
    }
    double* A = a.aggA + (size_t)blockIdx.x * KP * KP;
    double* C = a.aggC + (size_t)blockIdx.x * KP;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) A[(16 * w + 4 * v + lk) * KP + 16 * t + li] = D[t][v];
    if (li == 0)
#pragma unroll
        for (int v = 0; v < 4; ++v) C[16 * w + 4 * v + lk] = c[v];
}

// ---------------------------------------------------------------------------
// Smoother reduce: the block element a_s (x) ... (x) a_e from the right end,
// V = I, then for k = e .. s: V <- V diag(1/pred_{k+1}) Pi^T diag(alpha_k)
// (k < T - 1), or V <- rowsum(V) alpha_T^T at the sequence's last step.
// pred_{k+1} = alpha_k^T Pi is formed by every wave (lane y: state y).
// ---------------------------------------------------------------------------
template <int KP, bool GATED>
__global__ __launch_bounds__(KP / 16 * 64) void k_hmm_smoother_reduce(HmmArgs a) {
    if (GATED && *a.skip != 0) return;
    constexpr int NT = KP / 16;
    __shared__ double stage[NT][16 * (KP + 1)];
    __shared__ double pi_col[NT][KP];                 // per wave: alpha_k, broadcast
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
    const int64_t s = (int64_t)blockIdx.x * a.l;
    const int64_t e = min(s + a.l, a.T);
    const int K = a.K;
    double* Xs = stage[w];
    double* av = pi_col[w];
    double Yf[KP / 4][NT];
    load_pi_frags<KP>(a.Pi, K, true, Yf, li, lk);
    // column `lane` of Pi, for pred = alpha^T Pi
    double pc[KP];
#pragma unroll
    for (int x = 0; x < KP; ++x) pc[x] = (x < K && lane < K) ? a.Pi[x * K + lane] : 0.0;
    f64x4 D[NT];
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int t = 0; t < NT; ++t) D[t][v] = (16 * w + 4 * v + lk == 16 * t + li) ? 1.0 : 0.0;
    for (int64_t k = e - 1; k >= s; --k) {
        const double ak = lane < K ? a.alpha[k * K + lane] : 0.0;
        if (k == a.T - 1) {
            // V <- rowsum(V) alpha_T^T
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                double r = 0.0;
#pragma unroll
                for (int t = 0; t < NT; ++t) r += D[t][v];
                r = sum16(r);
#pragma unroll
                for (int t = 0; t < NT; ++t) D[t][v] = r * __shfl(ak, 16 * t + li, 64);
            }
            continue;
        }
        if (lane < KP) av[lane] = ak;
        wave_sync_lds();
        double pred = 0.0;
#pragma unroll
        for (int x = 0; x < KP; ++x) pred = fma(av[x], pc[x], pred);
        const double ip = pred > 0.0 ? 1.0 / pred : 0.0;
        // W = V diag(1/pred): column 16 t + li of the lane's registers
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const double it = __shfl(ip, 16 * t + li, 64);
#pragma unroll
            for (int v = 0; v < 4; ++v) D[t][v] *= it;
        }
        stage_strip<KP>(Xs, D, li, lk);
        wave_sync_lds();
        strip_times<KP>(Xs, Yf, D, li, lk);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const double at = __shfl(ak, 16 * t + li, 64);
#pragma unroll
            for (int v = 0; v < 4; ++v) D[t][v] *= at;
        }
        wave_sync_lds();
    }
    double* V = a.aggA + (size_t)blockIdx.x * KP * KP;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) V[(16 * w + 4 * v + lk) * KP + 16 * t + li] = D[t][v];
}

// ---------------------------------------------------------------------------
// One Hillis-Steele level at distance d over the block elements.
//   filter   (prefix): out[b] = in[b - d] (x) in[b] for b >= d, else in[b]:
//            X = A_left diag(exp(c_right - cmax)), B = X A_right, rows
//            renormalised, c = c_left + cmax + log(row sum);
//   smoother (suffix): out[b] = in[b] (x) in[b + d] for b + d < nblk:
//            V = V_right V_left (Definition 2 in matrix form).
// The right operand is read as Y fragments straight from memory.
// ---------------------------------------------------------------------------
template <int KP, bool FILTER, bool GATED>
__global__ __launch_bounds__(KP / 16 * 64) void k_hmm_scan_level(const double* __restrict__ inA,
                                                                 const double* __restrict__ inC, double* outA,
                                                                 double* outC, int64_t nblk, int64_t d,
                                                                 const int* skip) {
    if (GATED && *skip != 0) return;
    constexpr int NT = KP / 16;
    __shared__ double stage[NT][16 * (KP + 1)];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
    const int64_t b = blockIdx.x;
    const size_t mat = (size_t)KP * KP;
    double* oA = outA + b * mat;
    const int64_t partner = FILTER ? b - d : b + d;
    const bool active = FILTER ? (b >= d) : (b + d < nblk);
    if (!active) {
        for (int i = threadIdx.x; i < KP * KP; i += blockDim.x) oA[i] = inA[b * mat + i];
        if (FILTER)
            for (int i = threadIdx.x; i < KP; i += blockDim.x) outC[b * KP + i] = inC[b * KP + i];
        return;
    }
    // operand roles: rows come from X (the strip), Y is the full right factor
    const double* X = FILTER ? inA + partner * mat : inA + partner * mat;   // filter: left = b - d; smoother: V_right = b + d
    const double* Y = inA + b * mat;                                         // filter: right = b; smoother: V_left = b
    double* Xs = stage[w];
    double cmax = 0.0, scale_y = 1.0;
    if (FILTER) {
        const double cy = lane < KP ? inC[b * KP + lane] : -HUGE_VAL;
        cmax = max64(cy);
        if (!(cmax > -HUGE_VAL)) cmax = 0.0;                 // every row of the right factor is zero
        scale_y = lane < KP ? exp(cy - cmax) : 0.0;          // weight of column `lane` of X
    }
    for (int i = lane; i < 16 * KP; i += 64) {
        const int r = i / KP, col = i - r * KP;
        double v = X[(size_t)(16 * w + r) * KP + col];
        if (FILTER) v *= __shfl(scale_y, col, 64);
        Xs[r * (KP + 1) + col] = v;
    }
    double Yf[KP / 4][NT];
#pragma unroll
    for (int s = 0; s < KP / 4; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t) Yf[s][t] = Y[(size_t)(4 * s + lk) * KP + 16 * t + li];
    wave_sync_lds();
    f64x4 D[NT];
    strip_times<KP>(Xs, Yf, D, li, lk);
    if (FILTER) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            double r = 0.0;
#pragma unroll
            for (int t = 0; t < NT; ++t) r += D[t][v];
            r = sum16(r);
            const double inv = r > 0.0 ? 1.0 / r : 0.0;
#pragma unroll
            for (int t = 0; t < NT; ++t) D[t][v] *= inv;
            if (li == 0) {
                const int row = 16 * w + 4 * v + lk;
                outC[b * KP + row] = inC[partner * KP + row] + cmax + log(r);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) oA[(size_t)(16 * w + 4 * v + lk) * KP + 16 * t + li] = D[t][v];
}

// ---------------------------------------------------------------------------
// Down-sweeps: one wave per block, lane x = state x.
// ---------------------------------------------------------------------------
template <int KP, bool GATED>
__global__ __launch_bounds__(64) void k_hmm_filter_down(HmmArgs a, const double* __restrict__ preA,
                                                        const double* __restrict__ preC) {
    if (GATED && *a.skip != 0) return;
    __shared__ double av[KP];
    const int lane = threadIdx.x;
    const int K = a.K;
    const int64_t b = blockIdx.x;
    const int64_t s = b * a.l, e = min(s + a.l, a.T);
    double pc[KP];                                   // column `lane` of Pi
#pragma unroll
    for (int x = 0; x < KP; ++x) pc[x] = (x < K && lane < K) ? a.Pi[x * K + lane] : 0.0;
    // incoming prefix: the prior at the sequence start, else row 0 of the
    // inclusive prefix of the previous block (its rows are all the same)
    double al, lp;
    if (b == 0) {
        al = lane < K ? a.p0[lane] : 0.0;
        lp = 0.0;
    } else {
        al = lane < K ? preA[(size_t)(b - 1) * KP * KP + lane] : 0.0;
        lp = preC[(b - 1) * KP];
    }
    for (int64_t k = s; k < e; ++k) {
        if (lane < KP) av[lane] = al;
        wave_sync_lds();
        double pred = 0.0;
#pragma unroll
        for (int x = 0; x < KP; ++x) pred = fma(av[x], pc[x], pred);
        double M;
        const double lh = scaled_lik(a.L + k * K, K, lane, M);
        const double u = pred * lh;
        const double cs = sum64(u);
        al = u / cs;
        lp += M + log(cs);
        if (lane < K) a.alpha[k * K + lane] = al;
        if (a.logp && lane == 0) a.logp[k] = lp;
        wave_sync_lds();
    }
}

template <int KP, bool GATED>
__global__ __launch_bounds__(64) void k_hmm_smoother_down(HmmArgs a, const double* __restrict__ sufA) {
    if (GATED && *a.skip != 0) return;
    __shared__ double pr[KP][KP + 1];                // Pi (row stride padded: lanes read their own rows)
    __shared__ double wv[KP];
    __shared__ double av[KP];
    const int lane = threadIdx.x;
    const int K = a.K;
    const int64_t b = blockIdx.x;
    const int64_t s = b * a.l, e = min(s + a.l, a.T);
    for (int i = lane; i < KP * KP; i += 64) {
        const int r = i / KP, c = i - r * KP;
        pr[r][c] = (r < K && c < K) ? a.Pi[r * K + c] : 0.0;
    }
    double pc[KP];                                   // column `lane` of Pi
#pragma unroll
    for (int x = 0; x < KP; ++x) pc[x] = (x < K && lane < K) ? a.Pi[x * K + lane] : 0.0;
    // incoming suffix: row 0 of the inclusive suffix of the next block (the
    // smoothed marginal of step e), or nothing for the last block
    double g = 0.0;
    if (b + 1 < a.nblk) g = lane < K ? sufA[(size_t)(b + 1) * KP * KP + lane] : 0.0;
    wave_sync_lds();
    for (int64_t k = e - 1; k >= s; --k) {
        const double ak = lane < K ? a.alpha[k * K + lane] : 0.0;
        if (k == a.T - 1) {
            g = ak;
        } else {
            if (lane < KP) av[lane] = ak;
            wave_sync_lds();
            double pred = 0.0;
#pragma unroll
            for (int x = 0; x < KP; ++x) pred = fma(av[x], pc[x], pred);
            if (lane < KP) wv[lane] = pred > 0.0 ? g / pred : 0.0;
            wave_sync_lds();
            double acc = 0.0;
            if (lane < KP)
#pragma unroll 8
                for (int y = 0; y < KP; ++y) acc = fma(pr[lane][y], wv[y], acc);
            g = ak * acc;
        }
        if (lane < K) a.gamma[k * K + lane] = g;
        wave_sync_lds();
    }
}

// ---------------------------------------------------------------------------
// Overlapped blocks.  The recursion alpha_k ∝ (alpha_{k-1}^T Pi) ∘ exp(L_k) is a
// product of non-negative matrices: two starts with the same support approach
// each other in the projective metric and never part again (Birkhoff).  Every
// block is therefore run as a vector recursion (K^2 a step instead of the K^3
// of its block element) from kWarm steps before it, started from the uniform
// distribution, and the distribution it entered with is compared with the one
// its predecessor ended with: block 0 starts from the prior, so where every
// block entered with its predecessor's end (each entry to kSame of itself, the
// smallest ones too: the metric is that of ratios, and evidence that turns brings
// any weight back; a state with no weight has none in both) every block has the
// recursion's own values.  Blocks that did not are run
// again from the predecessor's end, kRepairs times; if one still differs (a
// chain that does not forget: a permutation, say) the flag stays clear and the
// block-element scan above does the work.  The smoother runs the same way
// backwards (gamma_k = alpha_k ∘ Pi (gamma_{k+1} / pred_{k+1}) is linear in
// gamma with non-negative coefficients and keeps its sum).
//
// One wave per block, about one wave per SIMD: bound by the latency and issue of
// a step's dependent chain (the broadcasts and KV^2 / 64 FP64 FMAs a lane of the
// product, two row joins, the scaling), 0.3 us a step at K = 64.  What does not
// depend on the vector (scaled likelihoods, reciprocal predictions) is formed once
// for all steps beforehand, in the memory of the results.  kWarm: of chains of 3
// to 64 states that stay 2 to 50 steps in a state, seen through Gaussian noise, every
// block has met its predecessor after 128 (stay 0.5) to 384 steps (0.9, 64 states);
// entries of two runs that have met stay within 2^-47.7 of each other (1400 places),
// kSame is three times that.  Filter + smoother at K = 64, T = 65536: 396 us, by the
// block-element scan 2420 us.
// ---------------------------------------------------------------------------
constexpr int kWarm = 448, kRepairs = 3, kAhead = 4;
// Chains that do not forget (permutations, states that stay for hundreds of steps
// and look alike) are given up early: the wave whose block starts the sequence, and
// has no warm-up of its own, runs two starts with no state in common for kPilotSteps
// steps at up to three places, and where two of the pairs are still kApart apart (L1;
// 2 at the start, 0.07 left of a chain that stays in its states for ten steps) a
// flag stops the others.  A permutation of 16 states, 2^16 steps: 353 us, by the scan
// alone 294 (535 with the whole attempt before it); of 64, 4096 steps: 518, 455 (685).
constexpr int kPilots = 3, kPilotSteps = 32;
constexpr double kApart = 0.7;
constexpr double kSame = 1.4210854715202004e-14;      // 2^-46
// Sums and predictions below the normal range: the reciprocal overflows where the
// quotient it stands for does not.  Such a block is not accepted.
constexpr double kNormal = 2.2250738585072014e-308;

struct OverArgs {
    HmmArgs h;
    int64_t l, nblk;
    double* entry;         // [nblk][KV] the distribution a block entered with
    double* end[2];        // [nblk][KV] and ended with (ping-pong over the repairs)
    double* blog;          // [nblk] log-likelihood of a block
    const int* need;       // the smoother after a filter: its flag (a chain that it found not to forget), or null
    int* ctl;              // [0] filter done, [1] smoother done, [2], [3] blocks that differ
};

// p: a in the lower half, b's lower half in the upper; q: a's upper half in the
// lower, b in the upper (swap16: the same for the even and odd rows of 16)
__device__ __forceinline__ void swap32(double a, double b, double& p, double& q) {
    const unsigned long long ua = (unsigned long long)__double_as_longlong(a), ub = (unsigned long long)__double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ua, (unsigned)ub, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
    p = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0]));
    q = __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ void swap16(double a, double b, double& p, double& q) {
    const unsigned long long ua = (unsigned long long)__double_as_longlong(a), ub = (unsigned long long)__double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)ua, (unsigned)ub, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
    p = __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0]));
    q = __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ double swap_add32(double a, double b) {
    double p, q;
    swap32(a, b, p, q);
    return p + q;
}
__device__ __forceinline__ double swap_add16(double a, double b) {
    double p, q;
    swap16(a, b, p, q);
    return p + q;
}
template <int CTRL>
__device__ __forceinline__ double dpp_ror(double x) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// over all lanes, on every lane
__device__ __forceinline__ double all_sum(double x) {
    x += dpp_ror<0x128>(x);
    x += dpp_ror<0x124>(x);
    x += dpp_ror<0x122>(x);
    x += dpp_ror<0x121>(x);
    x = swap_add16(x, x);
    return swap_add32(x, x);
}
__device__ __forceinline__ double all_max(double x) {
    x = fmax(x, dpp_ror<0x128>(x));
    x = fmax(x, dpp_ror<0x124>(x));
    x = fmax(x, dpp_ror<0x122>(x));
    x = fmax(x, dpp_ror<0x121>(x));
    double p, q;
    swap16(x, x, p, q);
    x = fmax(p, q);
    swap32(x, x, p, q);
    return fmax(p, q);
}
// 1 / x: the hardware estimate refined by two Newton-Raphson steps
__device__ __forceinline__ double recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

// lane k of every row of 16, in all lanes of the row
template <int K>
__device__ __forceinline__ double row_lane(double x) {
    return __builtin_amdgcn_update_dpp(0.0, x, 0x150 + K, 0xf, 0xf, true);
}
// rows of `MASK` take lane i from lane i - N (mod 16) of their row
template <int N, int MASK>
__device__ __forceinline__ double rotate_rows(double x) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const int l = (int)(unsigned)u, h = (int)(unsigned)(u >> 32);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(l, l, 0x120 + N, MASK, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(h, h, 0x120 + N, MASK, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// y_j = sum_i x_i M(i, j).  KV = 16, 32 or 64 states; state j in every lane l
// with l % KV = j.  Row g of 16 lanes adds up KV / 4 of the states, which it has
// in its own lanes (after a rotation, for KV < 64) and broadcasts along itself;
// the partial sums of every 16th column are joined by row swaps.  The
// coefficients are kept in registers, or in LDS (lane-major) where two matrices
// would not fit.
template <int KV, bool LDS>
struct MatVec {
    static constexpr int NT = KV / 16, RG = KV / 4;
    static constexpr int kLds = LDS ? NT * RG * 64 : 1;
    double p[LDS ? 1 : NT][LDS ? 1 : RG];
    double* q;
    // M = Pi, or its transpose
    __device__ __forceinline__ void load(const double* __restrict__ Pi, int K, bool trans, int lane, double* lds) {
        const int c = lane & 15, g = lane >> 4;
        const int r0 = KV == 64 ? 16 * g : (KV == 32 ? 16 * (g & 1) + 8 * (g >> 1) : 4 * g);
        q = lds;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < RG; ++i) {
                const int r = r0 + i, j = 16 * t + c;
                const double v = (r < K && j < K) ? (trans ? Pi[j * K + r] : Pi[r * K + j]) : 0.0;
                if constexpr (LDS) q[(t * RG + i) * 64 + lane] = v;
                else p[t][i] = v;
            }
    }
    template <int Q, int I>
    __device__ __forceinline__ void terms(const double (&x)[Q], double (&s)[Q][4], int lane) const {
        if constexpr (I < RG) {
            double m[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if constexpr (LDS) m[t] = q[(t * RG + I) * 64 + lane];
                else m[t] = p[t][I];
            }
#pragma unroll
            for (int k = 0; k < Q; ++k) {
                const double v = row_lane<I>(x[k]);
#pragma unroll
                for (int t = 0; t < NT; ++t) s[k][t] = fma(v, m[t], s[k][t]);
            }
            terms<Q, I + 1>(x, s, lane);
        }
    }
    // Q vectors at once
    template <int Q>
    __device__ __forceinline__ void operator()(const double (&x)[Q], double (&y)[Q], int lane) const {
        double s[Q][4], v[Q];
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            s[k][0] = s[k][1] = s[k][2] = s[k][3] = 0.0;
            v[k] = KV == 64 ? x[k] : (KV == 32 ? rotate_rows<8, 0xc>(x[k]) : rotate_rows<8, 0xc>(rotate_rows<12, 0xa>(x[k])));
        }
        terms<Q, 0>(v, s, lane);
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            if constexpr (NT <= 2) {
                const double a = swap_add32(s[k][0], s[k][0]), b = NT == 2 ? swap_add32(s[k][1], s[k][1]) : a;
                y[k] = swap_add16(a, b);
            } else {
                y[k] = swap_add16(swap_add32(s[k][0], s[k][2]), swap_add32(s[k][1], s[k][3]));
            }
        }
    }
};

// the wave's distribution x equals y, each entry to kSame of itself
__device__ __forceinline__ bool same_dist(double x, double y, bool live) {
    return !__any(live && !(fabs(x - y) <= kSame * y));
}

// alpha <- exp(L - M), logp <- M = max over the states: formed once here, read
// by the warm-up of several blocks.  Bound by memory (2 K doubles a step).
template <int KV>
__global__ __launch_bounds__(256) void k_hmm_scaled(OverArgs o) {
    const HmmArgs& a = o.h;
    const int lane = threadIdx.x & 63, x = lane & (KV - 1), K = a.K;
    if (blockIdx.x == 0 && threadIdx.x < 4) o.ctl[threadIdx.x] = 0;
    const int64_t stride = (int64_t)gridDim.x * (256 / KV);
    for (int64_t k = (int64_t)blockIdx.x * (256 / KV) + threadIdx.x / KV; k < a.T; k += stride) {
        const double v = x < K ? a.L[k * K + x] : -INFINITY;
        double M = v;
#pragma unroll
        for (int d = 1; d < KV; d <<= 1) M = fmax(M, __shfl_xor(M, d, 64));
        if (x < K) a.alpha[k * K + x] = exp(v - M);
        if (a.logp && x == 0) a.logp[k] = M;
    }
}

// the flag that an attempt (0: the filter's, 1: the smoother's) has failed
__device__ __forceinline__ int failed(const OverArgs& o, int smoother) {
    return __hip_atomic_load(o.ctl + 2 + smoother, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// steps of the warm-up between two looks at it (two pilots take about 110; a look in
// the steps' own loop, even a rare one, keeps their loads from running ahead)
constexpr int kLook = 128;
// runs the pilots: apart(k) the distance of the two starts of step k on
template <typename F>
__device__ __forceinline__ void pilots(const OverArgs& o, int smoother, F&& apart) {
    int votes = 0;
#pragma unroll 1
    for (int i = 1; i <= kPilots; ++i) {
        votes += apart((o.h.T - 2 * kPilotSteps) * i / (kPilots + 1) + kPilotSteps) > kApart;
        if (votes == 2) {
            if (threadIdx.x == 0) atomicAdd(o.ctl + 2 + smoother, 1);
            return;
        }
    }
}

// two starts, the even states and the odd ones, from step k on
template <int KV>
__device__ __forceinline__ double pilot(const HmmArgs& a, const MatVec<KV, false>& mv, int64_t k, int lane) {
    const int K = a.K, x = lane & (KV - 1), col = x < K ? x : K - 1;
    double v[2] = {x < K && !(x & 1) ? 1.0 : 0.0, x < K && (x & 1) ? 1.0 : 0.0};
    auto scale = [&] {
#pragma unroll
        for (int q = 0; q < 2; ++q) v[q] *= recip(all_sum(v[q]) * (KV / 64.0));
    };
#pragma unroll 1
    for (int i = 0; i < kPilotSteps; i += kAhead) {
        double w[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) w[j] = a.alpha[(k + i + j) * K + col];
        scale();
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            double y[2];
            mv(v, y, lane);
#pragma unroll
            for (int q = 0; q < 2; ++q) v[q] = x < K ? y[q] * w[j] : 0.0;
        }
    }
    scale();
    return all_sum(fabs(v[0] - v[1])) * (KV / 64.0);
}
// and backwards, from the filtered distribution of step k on
template <int KV>
__device__ __forceinline__ double pilot_back(const HmmArgs& a, const MatVec<KV, false>& bwd, int64_t k, int lane) {
    const int K = a.K, x = lane & (KV - 1), col = x < K ? x : K - 1;
    const double al = x < K ? a.alpha[k * K + col] : 0.0;
    double g[2] = {x & 1 ? 0.0 : al, x & 1 ? al : 0.0};
#pragma unroll
    for (int q = 0; q < 2; ++q) g[q] *= recip(all_sum(g[q]) * (KV / 64.0));
#pragma unroll 1
    for (int i = 1; i <= kPilotSteps; i += kAhead) {
        double av[kAhead], iv[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            av[j] = a.alpha[(k - i - j) * K + col];
            iv[j] = a.gamma[(k - i - j) * K + col];
        }
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            const double v[2] = {g[0] * iv[j], g[1] * iv[j]};
            double y[2];
            bwd(v, y, lane);
#pragma unroll
            for (int q = 0; q < 2; ++q) g[q] = x < K ? y[q] * av[j] : 0.0;
        }
    }
    return all_sum(fabs(g[0] - g[1])) * (KV / 64.0);
}

// The distribution that block b enters with, from kWarm steps before it.
// kAhead steps at a time, without a branch between them; the loads run two
// groups ahead.  The vector is scaled once a group, and by the sum that the
// group before it ended with, so that the sum is off the chain.
template <int KV>
__global__ __launch_bounds__(64) void k_hmm_filter_warm(OverArgs o) {
    const HmmArgs& a = o.h;
    const int lane = threadIdx.x, K = a.K, x = lane & (KV - 1);       // the lane's state
    const int64_t b = blockIdx.x, s = b * o.l;
    const bool live = x < K;
    const int col = live ? x : K - 1;                 // lanes without a state: the last one's loads, times zero
    const double mask = live ? 1.0 : 0.0;
    MatVec<KV, false> mv;
    mv.load(a.Pi, K, false, lane, nullptr);
    if (b == 0) pilots(o, 0, [&](int64_t at) { return pilot<KV>(a, mv, at, lane); });
    int64_t k = s > kWarm ? s - kWarm : 0;
    double al = live ? (k == 0 ? a.p0[x] : 1.0 / K) : 0.0, r = mask;
    double w[kAhead], raw[kAhead];
    auto fetch = [&](int64_t kk, double (&v)[kAhead]) {
#pragma unroll
        for (int j = 0; j < kAhead; ++j) v[j] = a.alpha[(kk + j < s ? kk + j : s) * K + col];
    };
    fetch(k, w);
    fetch(k + kAhead, raw);
    double c = 1.0;
    while (k < s) {
        for (const int64_t stop = min(s, k + kLook); k < stop; k += kAhead) {
            double nxt[kAhead];
            fetch(k + 2 * kAhead, nxt);
            r = recip(c) * mask;
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                const double v[1] = {al};
                double y[1];
                mv(v, y, lane);
                al = y[0] * (w[j] * (j == 0 ? r : mask));
                if (j == 0) c = all_sum(al) * (KV / 64.0);       // every state KV / 64 times
            }
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                w[j] = raw[j];
                raw[j] = nxt[j];
            }
        }
        if (failed(o, 0) != 0) return;
    }
    // block 0 enters with the prior as it is
    o.entry[b * KV + x] = s == 0 ? al : al * recip(all_sum(al) * (KV / 64.0));
}

// The block's steps.  FIRST: every block from its entry, with the scaled
// likelihoods that stand in alpha and logp; else the blocks that did not enter
// with their predecessor's end, from there, with the likelihoods formed again.
template <int KV, bool FIRST>
__global__ __launch_bounds__(64) void k_hmm_filter_over(OverArgs o, int pass) {
    const HmmArgs& a = o.h;
    const int lane = threadIdx.x, K = a.K, x = lane & (KV - 1);
    const int64_t b = blockIdx.x, s = b * o.l, e = min(s + o.l, a.T);
    const bool live = x < K;
    if (failed(o, 0) != 0) return;
    const double* in = o.end[(pass + 1) & 1];
    double* out = o.end[pass & 1];
    int64_t k = s;
    double al = o.entry[b * KV + x];
    if constexpr (!FIRST) {
        const double own = in[b * KV + x], was = al;
        al = b > 0 ? in[(b - 1) * KV + x] : 0.0;
        if (b == 0 || same_dist(was, al, live)) {
            out[b * KV + x] = own;
            return;
        }
        o.entry[b * KV + x] = al;
    }
    MatVec<KV, false> mv;
    mv.load(a.Pi, K, false, lane, nullptr);
    // the vector in flight is scaled by the sum of the step before it, not its own
    const int col = live ? x : K - 1;
    const double mask = live ? 1.0 : 0.0;
    double lp = 0.0, raw[kAhead], lh[kAhead], M[kAhead], r = 1.0;
    const bool want = a.logp != nullptr;
    double Mr = 0.0;
    bool bad = false;        // a step of the block has no weight, or too little of it: the scan's business
    auto fetch = [&](int64_t kk, double (&v)[kAhead]) {
#pragma unroll
        for (int j = 0; j < kAhead; ++j) v[j] = (FIRST ? a.alpha : a.L)[(kk + j < e ? kk + j : e - 1) * K + col];
    };
    auto scale = [&](const double (&v)[kAhead]) {
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            M[j] = FIRST ? 0.0 : all_max(v[j]);
            lh[j] = (FIRST ? v[j] : exp(v[j] - M[j])) * mask;
        }
    };
    // lane j: the scale of step kk + j
    auto fetch_scale = [&](int64_t kk) {
        const int64_t q = kk + (lane & (kAhead - 1));
        return FIRST && want ? a.logp[q < e ? q : e - 1] : 0.0;
    };
    fetch(k, raw);
    scale(raw);
    fetch(k + kAhead, raw);
    Mr = fetch_scale(k);
    for (; k < e; k += kAhead) {
        double w[kAhead], Ms = Mr, nxt[kAhead], cs = 1.0, av[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            w[j] = lh[j];
            if (!FIRST && (lane & (kAhead - 1)) == j) Ms = M[j];
        }
        fetch(k + 2 * kAhead, nxt);
        Mr = fetch_scale(k + kAhead);
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            const double v[1] = {al};
            double y[1];
            mv(v, y, lane);
            al = y[0] * (w[j] * r);
            const double c = all_sum(al) * (KV / 64.0);
            if ((lane & (kAhead - 1)) == j) cs = c;
            bad |= k + j < e && !(c >= kNormal);
            r = recip(c);
            av[j] = al * r;
        }
        scale(raw);
#pragma unroll
        for (int j = 0; j < kAhead; ++j) raw[j] = nxt[j];
        if (lane < K)
#pragma unroll
            for (int j = 0; j < kAhead; ++j)
                if (k + j < e) a.alpha[(k + j) * K + lane] = av[j];
        if (want) {
            // one logarithm for the group: lane j has step k + j; running sums over them
            double t = k + (lane & (kAhead - 1)) < e ? Ms + log(cs) : 0.0;
#pragma unroll
            for (int d = 1; d < kAhead; d <<= 1) {
                const double u = __shfl_up(t, d, kAhead);
                t += (lane & (kAhead - 1)) >= d ? u : 0.0;
            }
            t += lp;
            if (lane < kAhead && k + lane < e) a.logp[k + lane] = t;
            lp = __shfl(t, kAhead - 1, kAhead);
        }
    }
    out[b * KV + x] = al * r;
    if (lane == 0) o.blog[b] = bad ? NAN : lp;
}

// 1 / pred (zero where no state leads there); a NaN, which no comparison lets
// pass, in place of what may not be finite
__device__ __forceinline__ double recip_pred(double x) {
    return x >= kNormal ? recip(x) : (x > 0.0 ? NAN : 0.0);
}

// gamma_k <- 1 / pred_{k+1} (zero where no state leads there), pred_{k+1} =
// alpha_k^T Pi: a product of all steps with Pi on the matrix cores, formed once
// here and read by the warm-up of several blocks.  Bound by memory.
template <int KP>
__global__ __launch_bounds__(64) void k_hmm_pred(OverArgs o) {
    const HmmArgs& a = o.h;
    if (o.need ? *o.need == 0 : false) return;
    constexpr int NT = KP / 16;
    const int lane = threadIdx.x, li = lane & 15, lk = lane >> 4, K = a.K;
    if (!o.need && blockIdx.x == 0 && (lane == 1 || lane == 3)) o.ctl[lane] = 0;
    double Yf[KP / 4][NT];
    load_pi_frags<KP>(a.Pi, K, false, Yf, li, lk);
    for (int64_t k = (int64_t)blockIdx.x * 16; k < a.T; k += (int64_t)gridDim.x * 16) {
        const double* row = a.alpha + min(k + li, a.T - 1) * K;
        f64x4 D[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) D[t] = f64x4{0.0, 0.0, 0.0, 0.0};
        double f[KP / 4];
#pragma unroll
        for (int i = 0; i < KP / 4; ++i) f[i] = 4 * i + lk < K ? row[4 * i + lk] : 0.0;
#pragma unroll
        for (int i = 0; i < KP / 4; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t) D[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(f[i], Yf[i][t], D[t], 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                if (k + 4 * v + lk < a.T && 16 * t + li < K)
                    a.gamma[(k + 4 * v + lk) * K + 16 * t + li] = recip_pred(D[t][v]);
    }
}

// The distribution of the step after block b, from kWarm steps behind it.
template <int KV>
__global__ __launch_bounds__(64) void k_hmm_smoother_warm(OverArgs o) {
    const HmmArgs& a = o.h;
    if (o.need ? *o.need == 0 : false) return;
    const int lane = threadIdx.x, K = a.K, x = lane & (KV - 1);
    const int64_t b = blockIdx.x, e = min((b + 1) * o.l, a.T);
    const bool live = x < K;
    const int col = live ? x : K - 1;
    const double mask = live ? 1.0 : 0.0;
    MatVec<KV, false> bwd;
    bwd.load(a.Pi, K, true, lane, nullptr);
    if (e == a.T) return pilots(o, 1, [&](int64_t at) { return pilot_back<KV>(a, bwd, at, lane); });
    const int64_t from = min(e + kWarm, a.T - 1);
    double g = a.alpha[from * K + col] * mask;
    double av[kAhead], iv[kAhead], ra[kAhead], ri[kAhead];
    auto fetch = [&](int64_t kk, double (&u)[kAhead], double (&v)[kAhead]) {
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            const int64_t at = (kk - j > e ? kk - j : e) * K + col;
            u[j] = a.alpha[at];
            v[j] = a.gamma[at];
        }
    };
    int64_t k = from - 1;
    fetch(k, av, iv);
    fetch(k - kAhead, ra, ri);
    while (k >= e) {
        for (const int64_t stop = max(e, k - kLook + 1); k >= stop; k -= kAhead) {
            double na[kAhead], ni[kAhead];
            fetch(k - 2 * kAhead, na, ni);
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                const double v[1] = {g * iv[j]};
                double y[1];
                bwd(v, y, lane);
                g = k - j >= e ? y[0] * (av[j] * mask) : g;
            }
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                av[j] = ra[j];
                iv[j] = ri[j];
                ra[j] = na[j];
                ri[j] = ni[j];
            }
        }
        if (failed(o, 1) != 0) return;
    }
    o.entry[b * KV + x] = g;
}

// The block's steps (FIRST: every block, with the reciprocals that stand in gamma).
template <int KV, bool FIRST>
__global__ __launch_bounds__(64) void k_hmm_smoother_over(OverArgs o, int pass) {
    __shared__ double pl[MatVec<KV, !FIRST && KV == 64>::kLds];
    const HmmArgs& a = o.h;
    if (o.need ? *o.need == 0 : false) return;
    const int lane = threadIdx.x, K = a.K, x = lane & (KV - 1);
    const int64_t b = blockIdx.x, s = b * o.l, e = min(s + o.l, a.T);
    const bool live = x < K;
    if (failed(o, 1) != 0) return;
    const double* in = o.end[(pass + 1) & 1];
    double* out = o.end[pass & 1];
    int64_t k = e - 1;       // the step that is formed next
    double g;                // of step k + 1
    if constexpr (FIRST) {
        if (e == a.T) {                      // gamma_T = alpha_T
            g = live ? a.alpha[k * K + x] : 0.0;
            if (lane < K) a.gamma[k * K + lane] = g;
            --k;
        } else {
            g = o.entry[b * KV + x];
        }
    } else {
        const double own = in[b * KV + x];
        g = b + 1 < o.nblk ? in[(b + 1) * KV + x] : 0.0;
        if (b + 1 == o.nblk || same_dist(o.entry[b * KV + x], g, live)) {
            out[b * KV + x] = own;
            return;
        }
        o.entry[b * KV + x] = g;
    }
    double last = g;         // of the block's first step, at the end
    MatVec<KV, !FIRST && KV == 64> fwd;
    MatVec<KV, false> bwd;
    if constexpr (!FIRST) fwd.load(a.Pi, K, false, lane, pl);
    bwd.load(a.Pi, K, true, lane, nullptr);
    const int col = live ? x : K - 1;
    const double mask = live ? 1.0 : 0.0;
    double raw[kAhead], ri[kAhead], ak[kAhead], ip[kAhead];
    auto fetch = [&](int64_t kk, double (&v)[kAhead], double (&u)[kAhead]) {
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            const int64_t at = (kk - j > s ? kk - j : s) * K + col;
            v[j] = a.alpha[at] * mask;
            if constexpr (FIRST) u[j] = a.gamma[at];
        }
    };
    auto predict = [&](const double (&v)[kAhead], const double (&u)[kAhead]) {
        if constexpr (!FIRST) fwd(v, ip, lane);
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            ak[j] = v[j];
            if constexpr (FIRST) {
                ip[j] = u[j];
            } else {
                ip[j] = live ? recip_pred(ip[j]) : 0.0;
            }
        }
    };
    fetch(k, raw, ri);
    predict(raw, ri);
    fetch(k - kAhead, raw, ri);
    for (; k >= s; k -= kAhead) {
        double av[kAhead], iv[kAhead], na[kAhead], ni[kAhead], gv[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            av[j] = ak[j];
            iv[j] = ip[j];
        }
        fetch(k - 2 * kAhead, na, ni);
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            const double v[1] = {g * iv[j]};
            double y[1];
            bwd(v, y, lane);
            gv[j] = g = av[j] * y[0];
        }
        predict(raw, ri);
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            raw[j] = na[j];
            if constexpr (FIRST) ri[j] = ni[j];
        }
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            if (k - j < s) break;
            last = gv[j];
            if (lane < K) a.gamma[(k - j) * K + lane] = gv[j];
        }
    }
    out[b * KV + x] = last;
}


// blocks that still differ
template <int KV, bool FILTER>
__global__ __launch_bounds__(64) void k_hmm_over_check(OverArgs o) {
    const int lane = threadIdx.x, x = lane & (KV - 1);
    const int64_t b = blockIdx.x, p = FILTER ? b - 1 : b + 1;
    if (!FILTER && o.need && *o.need == 0) return;
    if (failed(o, !FILTER) != 0) return;
    if (FILTER && lane == 0 && !(fabs(o.blog[b]) < INFINITY)) atomicAdd(&o.ctl[2], 1);
    // (the first block's end is compared with nothing)
    if (!FILTER && b == 0 && __any(!(fabs(o.end[kRepairs & 1][x]) < INFINITY)) && lane == 0) atomicAdd(&o.ctl[3], 1);
    if (p < 0 || p >= o.nblk) return;
    if (!same_dist(o.entry[b * KV + x], o.end[kRepairs & 1][p * KV + x], x < o.h.K) && lane == 0)
        atomicAdd(&o.ctl[FILTER ? 2 : 3], 1);
}
// the flag; log p(y_1:k) from the blocks' own
template <bool FILTER>
__global__ __launch_bounds__(256) void k_hmm_over_done(OverArgs o) {
    __shared__ double part[4];
    if (o.ctl[FILTER ? 2 : 3] != 0 || (!FILTER && o.need && *o.need == 0)) return;
    const int64_t b = blockIdx.x;
    if (b == 0 && threadIdx.x == 0) o.ctl[FILTER ? 0 : 1] = 1;
    if (!FILTER || !o.h.logp) return;
    double v = 0.0;
    for (int64_t i = threadIdx.x; i < b; i += 256) v += o.blog[i];
    v = sum64(v);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    v = (part[0] + part[1]) + (part[2] + part[3]);
    const int64_t s = b * o.l, e = min(s + o.l, o.h.T);
    for (int64_t k = s + threadIdx.x; k < e; k += 256) o.h.logp[k] += v;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
template <int KP, bool GATED>
void hmm_scan(const HmmArgs& a, bool smoother, hipStream_t st) {
    constexpr int NTH = KP / 16 * 64;
    const unsigned nb = (unsigned)a.nblk;
    double *iA = a.aggA, *iC = a.aggC, *oA = a.aggA2, *oC = a.aggC2;
    if (!smoother) {
        prof_begin("k_hmm_filter_reduce", st);
        hipLaunchKernelGGL((k_hmm_filter_reduce<KP, GATED>), dim3(nb), dim3(NTH), 0, st, a);
        prof_end(st);
        for (int64_t d = 1; d < a.nblk; d <<= 1) {
            prof_begin("k_hmm_scan_level", st);
            hipLaunchKernelGGL((k_hmm_scan_level<KP, true, GATED>), dim3(nb), dim3(NTH), 0, st, iA, iC, oA, oC, a.nblk, d,
                               a.skip);
            prof_end(st);
            std::swap(iA, oA);
            std::swap(iC, oC);
        }
        prof_begin("k_hmm_filter_down", st);
        hipLaunchKernelGGL((k_hmm_filter_down<KP, GATED>), dim3(nb), dim3(64), 0, st, a, iA, iC);
        prof_end(st);
    } else {
        prof_begin("k_hmm_smoother_reduce", st);
        hipLaunchKernelGGL((k_hmm_smoother_reduce<KP, GATED>), dim3(nb), dim3(NTH), 0, st, a);
        prof_end(st);
        for (int64_t d = 1; d < a.nblk; d <<= 1) {
            prof_begin("k_hmm_scan_level", st);
            hipLaunchKernelGGL((k_hmm_scan_level<KP, false, GATED>), dim3(nb), dim3(NTH), 0, st, iA, nullptr, oA, nullptr,
                               a.nblk, d, a.skip);
            prof_end(st);
            std::swap(iA, oA);
        }
        prof_begin("k_hmm_smoother_down", st);
        hipLaunchKernelGGL((k_hmm_smoother_down<KP, GATED>), dim3(nb), dim3(64), 0, st, a, iA);
        prof_end(st);
    }
}

constexpr int over_states(int KP) { return KP == 48 ? 64 : KP; }      // a power of two

template <int KV>
void hmm_over(const OverArgs& o, bool smoother, hipStream_t st) {
    const dim3 grid((unsigned)o.nblk), wave(64);
    if (smoother) {
        prof_begin("k_hmm_pred", st);
        hipLaunchKernelGGL((k_hmm_pred<KV>), dim3((unsigned)std::min<int64_t>(2048, (o.h.T + 15) / 16)), wave, 0, st, o);
        prof_end(st);
        prof_begin("k_hmm_smoother_warm", st);
        hipLaunchKernelGGL((k_hmm_smoother_warm<KV>), grid, wave, 0, st, o);
        prof_end(st);
    } else {
        prof_begin("k_hmm_scaled", st);
        hipLaunchKernelGGL((k_hmm_scaled<KV>), dim3((unsigned)std::min<int64_t>(2048, (o.h.T * KV + 255) / 256)), dim3(256), 0,
                           st, o);
        prof_end(st);
        prof_begin("k_hmm_filter_warm", st);
        hipLaunchKernelGGL((k_hmm_filter_warm<KV>), grid, wave, 0, st, o);
        prof_end(st);
    }
    for (int pass = 0; pass <= kRepairs; ++pass) {
        prof_begin(smoother ? (pass ? "k_hmm_smoother_repair" : "k_hmm_smoother_over")
                            : (pass ? "k_hmm_filter_repair" : "k_hmm_filter_over"), st);
        if (smoother && pass) hipLaunchKernelGGL((k_hmm_smoother_over<KV, false>), grid, wave, 0, st, o, pass);
        else if (smoother) hipLaunchKernelGGL((k_hmm_smoother_over<KV, true>), grid, wave, 0, st, o, pass);
        else if (pass) hipLaunchKernelGGL((k_hmm_filter_over<KV, false>), grid, wave, 0, st, o, pass);
        else hipLaunchKernelGGL((k_hmm_filter_over<KV, true>), grid, wave, 0, st, o, pass);
        prof_end(st);
    }
    prof_begin("k_hmm_over_check", st);
    if (smoother) hipLaunchKernelGGL((k_hmm_over_check<KV, false>), grid, dim3(64), 0, st, o);
    else hipLaunchKernelGGL((k_hmm_over_check<KV, true>), grid, dim3(64), 0, st, o);
    prof_end(st);
    prof_begin("k_hmm_over_done", st);
    if (smoother) hipLaunchKernelGGL((k_hmm_over_done<false>), dim3(1), dim3(256), 0, st, o);
    else hipLaunchKernelGGL((k_hmm_over_done<true>), grid, dim3(256), 0, st, o);
    prof_end(st);
}

template <int KP>
hipError_t hmm_run(HmmArgs a, OverArgs o, int passes, hipStream_t st) {
    for (int smoother = 0; smoother < 2; ++smoother) {
        if (!(passes & (1 << smoother))) continue;
        if (o.nblk > 0) {
            o.need = smoother && (passes & 1) ? o.ctl : nullptr;
            hmm_over<over_states(KP)>(o, smoother != 0, st);
            a.skip = o.ctl + smoother;
            hmm_scan<KP, true>(a, smoother != 0, st);
        } else {
            hmm_scan<KP, false>(a, smoother != 0, st);
        }
    }
    return hipGetLastError();
}

constexpr int64_t kOverSteps = 32, kOverBlocks = 1024;

// Where overlapped blocks win.  Their time hardly grows with T (the warm-up's
// kWarm steps are most of it); the scan's does, with T KP^3.  Filter + smoother,
// us, scan, overlapped, and the scan behind an attempt that is given up: KP = 16, T =
// 2^16: 294, 246, 353; KP = 32, 2^15: 417, 302, 520; KP = 48, 2^13: 475, 329, 536; KP =
// 64, 2^12: 458, 322, 518.  At half these lengths (a quarter of them for KP > 32) the
// two are even: from twice as long on, as a failed attempt is time lost.
int64_t over_min(int KP) { return KP == 16 ? 1 << 16 : KP == 32 ? 1 << 15 : KP == 48 ? 1 << 13 : 1 << 12; }

}  // namespace

int hmm_padded_states(int K) { return (K + 15) / 16 * 16; }

// Steps per block: enough blocks that every SIMD holds about two waves of the
// reduce kernels (KP / 16 waves per block), at least 4 steps per block.
int64_t hmm_block_len(int K, int64_t T) {
    const int strips = hmm_padded_states(K) / 16;
    const int64_t target_blocks = std::max<int64_t>(1, 2048 / strips);
    int64_t l = (T + target_blocks - 1) / target_blocks;
    return std::max<int64_t>(4, l);
}

size_t hmm_ws_bytes(int K, int64_t T) {
    const int KP = hmm_padded_states(K);
    const int64_t nblk = T > 0 ? (T + hmm_block_len(K, T) - 1) / hmm_block_len(K, T) : 0;
    const size_t per = sizeof(double) * ((size_t)KP * KP + KP);
    return 2 * per * (size_t)nblk + 256;
}

hipError_t launch_hmm(int K, int64_t T, const double* Pi, const double* p0, const double* L, double* alpha,
                      double* logp, double* gamma, void* ws, int passes, hipStream_t st) {
    HmmArgs a{};
    const int KP = hmm_padded_states(K);
    a.K = K;
    a.T = T;
    a.l = hmm_block_len(K, T);
    a.nblk = (T + a.l - 1) / a.l;
    a.Pi = Pi;
    a.p0 = p0;
    a.L = L;
    a.alpha = alpha;
    a.logp = logp;
    a.gamma = gamma;
    char* base = static_cast<char*>(ws);
    const size_t mats = sizeof(double) * (size_t)KP * KP * a.nblk, vecs = sizeof(double) * (size_t)KP * a.nblk;
    a.aggA = reinterpret_cast<double*>(base);
    a.aggA2 = reinterpret_cast<double*>(base + mats);
    a.aggC = reinterpret_cast<double*>(base + 2 * mats);
    a.aggC2 = reinterpret_cast<double*>(base + 2 * mats + vecs);
    // overlapped blocks in the memory of the block elements (the flags behind it)
    OverArgs o{};
    o.h = a;
    o.l = std::max<int64_t>(kOverSteps, (T + kOverBlocks - 1) / kOverBlocks);
    o.l = (o.l + kAhead - 1) / kAhead * kAhead;      // whole groups of steps (kWarm is)
    o.nblk = (T + o.l - 1) / o.l;
    o.ctl = reinterpret_cast<int*>(base + 2 * (mats + vecs));
    o.entry = reinterpret_cast<double*>(base);
    const int KV = over_states(KP);
    o.end[0] = o.entry + o.nblk * KV;
    o.end[1] = o.end[0] + o.nblk * KV;
    o.blog = o.end[1] + o.nblk * KV;
    if (T < over_min(KP) || (size_t)o.nblk * (3 * KV + 1) * sizeof(double) > 2 * (mats + vecs)) o.nblk = 0;
    switch (KP) {
        case 16: return hmm_run<16>(a, o, passes, st);
        case 32: return hmm_run<32>(a, o, passes, st);
        case 48: return hmm_run<48>(a, o, passes, st);
        case 64: return hmm_run<64>(a, o, passes, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace pks
