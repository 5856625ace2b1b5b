// steady.hpp -- filter and smoother of time-invariant models whose covariances
// converge (one sequence, or packed sequences of one shared model).
//
// The covariances of a time-invariant model do not depend on the
// measurements, and for a model the filter can follow they settle: the block
// element of n steps (Lemma 2 applied to equal elements) has P_k = A X A^T + C
// with X <= P_{k-n}, so once the remainder A X A^T is below the rounding of C
// every later filtered covariance is C to FP64's rounding.  Below it means entry
// by entry: the remainder is positive semidefinite, so that its entry (i, j) is at
// most the root of the product of two of its diagonal, and each of those is held
// against the variance of its own state (states of different units, or one that
// is hardly driven, have variances many orders apart).  The same holds
// for the smoothing element (Lemma 4): Ps_k = E^n Ps_{k+n} E^nT + L.  The
// setup finds the smallest such power of two n by recursive doubling (a chain
// of log2 n combines instead of one O(nx^3) combine per step), forms
//   the first n filtered covariances and gains (from the prior),
//   the first n smoothed covariances (from the settled one, backwards) and
//   the last n smoothed covariances (from the last filtered one, backwards),
// and everything else is the settled value.  What is left per step is the
// affine recursion of the means,
//   m_k  = Phi_k m_{k-1} + K_k y_k + c_k          (Phi = (I - K H) F),
//   ms_k = m_k + E_k (ms_{k+1} - F m_k - u),
// scanned over blocks of L steps (Section III-C) with the constant matrices
// Phi^L, E^L beyond the head.  A model that does not settle within the table's
// N steps leaves the flag ctl[0] at zero, and the general scan kernels, which
// follow in the stream and return at once when the flag is set, do the work.
// The smoother alone (nx > 16) compares every filtered covariance that it is
// given with the table's, in the storage type: they are those of the filter
// here, or the general kernels take the call.
#pragma once
#include "pks_internal.h"

namespace pks {
namespace steady {

constexpr int kRun = 4;              // steps a wave takes from each doubled start (tables)
constexpr int kBlockChains = 64;     // chains of a workgroup of four waves
constexpr int kPowers = 11;          // L .. 1024 L

struct Args {
    int nx, ny, B;
    int N;                       // longest head the tables hold (a power of two)
    int pL;                      // log2 of the steps per chain
    int smooth;                  // filter + smoother (else the filter alone)
    int given;                   // the smoother alone, of filtered moments that the call has
    int reset;
    int64_t total;
    const int64_t* offsets;      // device [B+1]; nullptr: one sequence
    const double *F, *u, *Q, *H, *d, *R, *m0, *P0;
    const void* y;
    void *m, *P, *ms, *Ps;
    int* status;
    int* ctl;                    // [0] n (0: not settled), [1] log2 of the filter's n, [2] of the smoother's
    int64_t* blk_off;            // [B+1] chain blocks of the sequences before
    double* star;                // settled P, Phi, E, L, Ps, K, c
    double *powF, *powE;         // [levels][3 n^2] A, C, J; [levels][2 n^2] E, L of 2^l steps
    double *mpF, *mpE;           // [kPowers][n^2] Phi^(L 2^i), E^(L 2^i)
    double *tP, *tPhi, *tK, *tc, *tE, *tL, *tHead, *tTail;     // [N] tables
    double *runPhi, *runE, *runL, *runC;   // [N / kRun] of a run: Phi, smoothing element, smoothed covariance that enters
    double *scanE[2], *scanL[2];           // nx > 16: suffix scan of the runs' smoothing elements
    double *pre, *agg, *car;     // [chains][n], [blocks][n]: what chains and blocks add, what enters blocks
    double *runB, *runX;         // [B][N / kRun][n]: what a run of a head adds, what enters it
    int64_t max_blocks;
};

__host__ __device__ inline int64_t star_words(int n, int m) { return 5 * (int64_t)n * n + (int64_t)n * m + n; }
__host__ __device__ inline int64_t star_P(int, int) { return 0; }
__host__ __device__ inline int64_t star_Phi(int n, int) { return (int64_t)n * n; }
__host__ __device__ inline int64_t star_E(int n, int) { return 2 * (int64_t)n * n; }
__host__ __device__ inline int64_t star_L(int n, int) { return 3 * (int64_t)n * n; }
__host__ __device__ inline int64_t star_Ps(int n, int) { return 4 * (int64_t)n * n; }
__host__ __device__ inline int64_t star_K(int n, int) { return 5 * (int64_t)n * n; }
__host__ __device__ inline int64_t star_c(int n, int m) { return 5 * (int64_t)n * n + (int64_t)n * m; }

// whether the call may take this path (sizes alone), and its workspace layout:
// fills the pointers of `a` inside [base, base + bytes); false: does not fit
bool applies(int nx, int ny, int32_t B, int64_t total, bool mixed);
bool layout(Args& a, char* base, size_t bytes);
hipError_t launch(Args a, bool mixed, hipStream_t s);
hipError_t launch_large(const Args& a, bool mixed, hipStream_t s);       // 16 < nx <= 64

}  // namespace steady
}  // namespace pks
