// steady_ops.hpp -- shared by the two sizes of the settled-covariance path
// (steady.hip: nx <= 16, steady_large.hip: 16 < nx <= 64): register-tile
// primitives, packed sequences, and the covariance rows of all steps.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "steady.hpp"
#include "tile16.hpp"

namespace pks {
namespace steady {

using namespace w16;

// how small each variance of A (P0 + C) A^T has to be against C's: FP64 rounding
// with 2^7 to spare for covariances of the head above the prior and the settled
// one (checked when the head is formed)
constexpr double kTiny = 8.673617379884035e-19;      // 2^-60
constexpr double kSpare = 128.0;
// Residuals, in every entry, of an inverse formed without row exchanges: rounding
// (1e-15 where no pivot is small), and what one Newton step still brings there.  (Kept
// as it was at a residual of 1e-11, the settled covariance of a model with a pivot
// of 1e-3 was 1.7e-13 off; 7e-16 after the step.)
constexpr double kExact = 1e-14, kSmall = 1e-8;
// and how far the last covariance of the head (the tail), which is formed step by
// step, may be from the settled one, which is doubled: two digits inside the parity bar
constexpr double kMeet = 1e-11;

// ---------------------------------------------------------------------------
// tiles with KX (KY) K-slices: rows and columns beyond 4 KX are zero
// ---------------------------------------------------------------------------
// columns moved by D (zero enters): lane i takes lane i - D (up) or i + D (down) of its row of 16
template <int CTRL>
__device__ __forceinline__ double dpp0(double x) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <bool UP, int D, int KX>
__device__ __forceinline__ f64x4 shift(const f64x4& x) {
    f64x4 t = zero4();
#pragma unroll
    for (int v = 0; v < KX; ++v) t[v] = UP ? dpp0<0x110 + D>(x[v]) : dpp0<0x100 + D>(x[v]);
    return t;
}

// tiles: each diagonal entry of x is at most f times y's (the first n)
__device__ __forceinline__ bool diagonal_below(const f64x4& x, const f64x4& y, double f, int n) {
    const int li = lane_i(), lk = lane_k();
    bool off = false;
#pragma unroll
    for (int v = 0; v < 4; ++v) off |= 4 * v + lk == li && li < n && !(x[v] <= f * y[v]);
    return !__any(off);
}
// x equals y, each entry to kMeet of the root of the product of its variances (di,
// dj: those of y along the rows and the columns)
__device__ __forceinline__ bool meets(const f64x4& x, const f64x4& y, const f64x4& di, const f64x4& dj) {
    bool off = false;
#pragma unroll
    for (int v = 0; v < 4; ++v) off |= !((x[v] - y[v]) * (x[v] - y[v]) <= kMeet * kMeet * (di[v] * dj[v]));
    return !__any(off);
}
__device__ __forceinline__ f64x4 diagonal(const f64x4& x) {
    const int li = lane_i(), lk = lane_k();
    f64x4 t;
#pragma unroll
    for (int v = 0; v < 4; ++v) t[v] = 4 * v + lk == li ? x[v] : 0.0;
    return t;
}
__device__ __forceinline__ f64x4 ones() { return f64x4{1.0, 1.0, 1.0, 1.0}; }

// Inverse by Gauss-Jordan elimination without pivoting, as w16::inv_diag, with
// a constant number NP of pivots (rows beyond the matrix hold the identity), so
// that no branch keeps the compiler from overlapping it with other work.
template <int NP, bool SPD>
__device__ __forceinline__ f64x4 inv_np(f64x4 a, bool& ok) {
    const int li = lane_i(), lk = lane_k();
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const int q = k >> 2, g = k & 3;
        const double pv = readlane_d(a[q], (g << 4) | k);
        double ck[4];
#pragma unroll
        for (int v = 0; v < NP / 4; ++v) ck[v] = col_bcast(a[v], k);
        const double rk = row_bcast(a[q], g);
        ok = ok && (SPD ? pv > 0.0 : pv != 0.0) && isfinite(pv);
        const double r = recip(pv);
        const double rr = rk * r;
#pragma unroll
        for (int v = 0; v < NP / 4; ++v) {
            const double f = ck[v] * r;
            if (4 * v + lk == k) a[v] = li == k ? r : rr;
            else a[v] = li == k ? -f : fma(-f, rk, a[v]);
        }
    }
    return a;
}

// ---------------------------------------------------------------------------
// sequences
// ---------------------------------------------------------------------------
struct SeqR {
    int b;
    int64_t start, end;
};
__device__ __forceinline__ SeqR seq_of(const Args& a, int b) {
    if (!a.offsets) return SeqR{0, 0, a.total};
    return SeqR{b, a.offsets[b], a.offsets[b + 1]};
}
__device__ __forceinline__ int seq_holding(const int64_t* off, int B, int64_t k) {     // off[b] <= k < off[b + 1]
    int lo = 0, hi = B;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= k) lo = mid; else hi = mid;
    }
    return lo;
}

// ---------------------------------------------------------------------------
// covariance rows of all steps, from the tables, by the workgroups of a launch
// that are left (wg of nwg).  Bound by the HBM writes: consecutive threads on
// consecutive 16-byte units of a contiguous range of rows, streaming stores;
// the settled row comes from LDS.
// ---------------------------------------------------------------------------
template <typename R, int BYTES> struct Unit;
template <typename R> struct Unit<R, 16> { using T = unsigned __attribute__((ext_vector_type(4))); };
template <typename R> struct Unit<R, 8> { using T = unsigned __attribute__((ext_vector_type(2))); };
template <typename R> struct Unit<R, 4> { using T = unsigned; };

// CHECK: compares the rows that are there instead; true if one differs
template <typename R, int BYTES, bool SMOOTHED, bool CHECK>
__device__ __forceinline__ bool write_rows_u(const Args& a, int nh, int64_t wg, int64_t nwg, R* lds) {
    using UT = typename Unit<R, BYTES>::T;
    constexpr int V = BYTES / (int)sizeof(R);
    const int n = a.nx, n2 = n * n;
    const double* settled = a.star + (SMOOTHED ? star_Ps(n, a.ny) : star_P(n, a.ny));
    for (int i = threadIdx.x; i < n2; i += blockDim.x) lds[i] = R(settled[i]);
    __syncthreads();
    R* dst = static_cast<R*>(SMOOTHED ? a.Ps : a.P);
    const int upr = n2 / V, S = blockDim.x;
    const int64_t per = (a.total + nwg - 1) / nwg;
    const int64_t r0 = wg * per, r1 = r0 + per < a.total ? r0 + per : a.total;
    int64_t row = r0 + threadIdx.x / upr;
    int off = threadIdx.x % upr;
    const int srow = S / upr, soff = S % upr;
    bool differs = false;
    if (row >= r1) return false;
    int b = a.offsets ? seq_holding(a.offsets, a.B, row) : 0;
    SeqR q = seq_of(a, b);
    UT* out = reinterpret_cast<UT*>(dst);
    while (row < r1) {
        while (row >= q.end) q = seq_of(a, q.b + 1);
        const int64_t k = row - q.start, len = q.end - q.start;
        UT v;
        bool mine = true;
        const double* src = nullptr;
        if (!SMOOTHED) {
            if (k < nh - 1) src = a.tP + k * n2;
        } else if (len < 2 * nh && k < nh - 1) {
            mine = false;                        // a short sequence's head is its own (short_head)
        } else if (k < nh - 1) {
            src = a.tHead + k * n2;
        } else if (len - 1 - k < nh - 1) {
            src = a.tTail + (len - 1 - k) * n2;
        }
        if (src) {
            R t[V];
#pragma unroll
            for (int i = 0; i < V; ++i) t[i] = R(src[off * V + i]);
            __builtin_memcpy(&v, t, BYTES);
        } else {
            __builtin_memcpy(&v, lds + off * V, BYTES);
        }
        if constexpr (CHECK) {
            const UT x = out[row * upr + off];
            unsigned vw[BYTES / 4], xw[BYTES / 4];
            __builtin_memcpy(vw, &v, BYTES);
            __builtin_memcpy(xw, &x, BYTES);
#pragma unroll
            for (int i = 0; i < BYTES / 4; ++i) differs |= vw[i] != xw[i];
        } else if (mine) {
            __builtin_nontemporal_store(v, out + row * upr + off);
        }
        row += srow;
        off += soff;
        if (off >= upr) {
            off -= upr;
            ++row;
        }
    }
    return differs;
}
template <typename R, bool SMOOTHED>
__device__ __forceinline__ void write_rows(const Args& a, int nh, int64_t wg, int64_t nwg, R* lds) {
    if ((a.nx & 1) == 0) write_rows_u<R, 16, SMOOTHED, false>(a, nh, wg, nwg, lds);
    else write_rows_u<R, sizeof(R), SMOOTHED, false>(a, nh, wg, nwg, lds);
}
template <typename R>
__device__ __forceinline__ bool rows_differ(const Args& a, int nh, int64_t wg, int64_t nwg, R* lds) {
    return (a.nx & 1) == 0 ? write_rows_u<R, 16, false, true>(a, nh, wg, nwg, lds)
                           : write_rows_u<R, sizeof(R), false, true>(a, nh, wg, nwg, lds);
}

// column of a tile <-> vector of n in memory
template <int KX, typename T>
__device__ __forceinline__ f64x4 load_col(const T* x, int n) {
    const int lk = lane_k();
    f64x4 t = zero4();
#pragma unroll
    for (int v = 0; v < KX; ++v)
        if (4 * v + lk < n) t[v] = double(x[4 * v + lk]);
    return t;
}
template <int KX, typename T>
__device__ __forceinline__ void store_col(T* x, const f64x4& t, int n) {
    const int lk = lane_k();
#pragma unroll
    for (int v = 0; v < KX; ++v)
        if (4 * v + lk < n) x[4 * v + lk] = T(t[v]);
}
// operand of a product with the n x m matrix X from the left: the tile of X^T
template <int KX>
__device__ __forceinline__ f64x4 load_op(const double* X, int n, int m) {
    const int li = lane_i(), lk = lane_k();
    f64x4 t = zero4();
#pragma unroll
    for (int v = 0; v < KX; ++v)
        if (li < n && 4 * v + lk < m) t[v] = X[li * m + 4 * v + lk];
    return t;
}

// the sequence of this lane's column in a group of 16 (heads)
struct Head {
    int64_t start;
    int len, b;            // steps, at most nh (0: no sequence)
    int64_t full;
};
__device__ __forceinline__ Head head_of(const Args& a, int nh, int group) {
    Head h;
    h.b = group * 16 + lane_i();
    const bool live = h.b < a.B;
    if (!live) h.b = a.B - 1;
    const SeqR q = seq_of(a, h.b);
    h.start = q.start;
    h.full = live ? q.end - q.start : 0;
    h.len = (int)(h.full < nh ? h.full : nh);
    return h;
}
__device__ __forceinline__ double* run_vec(const Args& a, double* base, int b, int run) {
    return base + ((int64_t)b * (a.N / kRun) + run) * a.nx;
}

}  // namespace steady
}  // namespace pks
