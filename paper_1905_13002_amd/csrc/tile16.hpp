// tile16.hpp -- matrices of up to 16 x 16 in the registers of one wavefront:
// layout, products, transposes and inverses shared by the register-resident
// scans (scan_w16.hip) and the converged-covariance path (steady.hip).
//
// Register layout of a 16 x 16 matrix X (smaller dimensions padded with
// zeros): lane l = 16 lk + li holds X(4 v + lk, li) in component v of an
// f64x4 -- the accumulator layout of v_mfma_f64_16x16x4f64.  In that layout
// component s of the tile of L^T and component s of the tile of R are
// exactly the A and B operands of the s-th K-slice of the product L R, so a
// product is four MFMAs with no data movement:
//     L R = mm(tile(L^T), tile(R)),   (L R)^T = mm(tile(R), tile(L^T)).
// A vector x is held replicated across the columns (lane: x(4 v + lk)).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace pks {
namespace w16 {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 256;                    // doubles of one tile in memory (lane-major)
constexpr int kStage = 16 * 17;               // LDS doubles per wave: the row gather of a pivoted inverse
constexpr int kThreads = 64;

__device__ __forceinline__ int lane_i() { return threadIdx.x & 15; }          // column
__device__ __forceinline__ int lane_k() { return (threadIdx.x >> 4) & 3; }    // row within a group of four

__device__ __forceinline__ f64x4 zero4() { return f64x4{0.0, 0.0, 0.0, 0.0}; }

__device__ __forceinline__ f64x4 eye() {
    const int li = lane_i(), lk = lane_k();
    f64x4 t;
#pragma unroll
    for (int v = 0; v < 4; ++v) t[v] = (4 * v + lk == li) ? 1.0 : 0.0;
    return t;
}

// L R + acc, given the tile of L^T and the tile of R.  KS: the K-slices of four
// that hold the contraction (entries beyond 4 KS of L's columns or R's rows
// are zero), so a contraction over ny <= 8 takes two MFMAs; a compile-time
// count, since a branch around each MFMA costs more than the MFMA
template <int KS = 4>
__device__ __forceinline__ f64x4 mm(const f64x4& lt, const f64x4& r, f64x4 acc) {
#pragma unroll
    for (int s = 0; s < KS; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(lt[s], r[s], acc, 0, 0, 0);
    return acc;
}
template <int KS = 4>
__device__ __forceinline__ f64x4 mm(const f64x4& lt, const f64x4& r) { return mm<KS>(lt, r, zero4()); }

// (X + X^T) / 2 + add, given the tiles of X and X^T
__device__ __forceinline__ f64x4 sym(const f64x4& x, const f64x4& xt, const f64x4& add) {
    f64x4 t;
#pragma unroll
    for (int v = 0; v < 4; ++v) t[v] = 0.5 * (x[v] + xt[v]) + add[v];
    return t;
}

// ---------------------------------------------------------------------------
// memory <-> registers
// ---------------------------------------------------------------------------
// tile of the rows x cols matrix X (row stride ld), zero outside it
template <typename T>
__device__ __forceinline__ f64x4 load_tile(const T* X, int rows, int cols, int ld) {
    const int li = lane_i(), lk = lane_k();
    f64x4 t;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = 4 * v + lk;
        t[v] = (r < rows && li < cols) ? double(X[r * ld + li]) : 0.0;
    }
    return t;
}
// tile of X^T for the rows x cols matrix X
template <typename T>
__device__ __forceinline__ f64x4 load_tile_t(const T* X, int rows, int cols, int ld) {
    const int li = lane_i(), lk = lane_k();
    f64x4 t;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = 4 * v + lk;
        t[v] = (li < rows && r < cols) ? double(X[li * ld + r]) : 0.0;
    }
    return t;
}
// replicated vector x[0..n), zero beyond
template <typename T>
__device__ __forceinline__ f64x4 load_vec(const T* x, int n) {
    const int lk = lane_k();
    f64x4 t;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = 4 * v + lk;
        t[v] = r < n ? double(x[r]) : 0.0;
    }
    return t;
}
template <typename T>
__device__ __forceinline__ void store_tile(T* X, const f64x4& t, int n) {
    const int li = lane_i(), lk = lane_k();
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = 4 * v + lk;
        if (r < n && li < n) X[r * n + li] = T(t[v]);
    }
}
template <typename T>
__device__ __forceinline__ void store_vec(T* x, const f64x4& t, int n) {
    const int li = lane_i(), lk = lane_k();
    if (li != 0) return;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = 4 * v + lk;
        if (r < n) x[r] = T(t[v]);
    }
}
// records: tiles lane-major (each lane's four doubles contiguous)
__device__ __forceinline__ void put_tile(double* p, const f64x4& t) {
    reinterpret_cast<f64x4*>(p)[threadIdx.x & 63] = t;
}
__device__ __forceinline__ f64x4 get_tile(const double* p) {
    return reinterpret_cast<const f64x4*>(p)[threadIdx.x & 63];
}

__device__ __forceinline__ double readlane_d(double x, int l) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// lane k of the lane's own row of 16 (DPP row_newbcast; k a constant after unrolling)
__device__ __forceinline__ unsigned newbcast(unsigned x, int k) {
    switch (k) {
#define PKS_NB(K) case K: return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x150 + K, 0xf, 0xf, false);
        PKS_NB(0) PKS_NB(1) PKS_NB(2) PKS_NB(3) PKS_NB(4) PKS_NB(5) PKS_NB(6) PKS_NB(7)
        PKS_NB(8) PKS_NB(9) PKS_NB(10) PKS_NB(11) PKS_NB(12) PKS_NB(13) PKS_NB(14) PKS_NB(15)
#undef PKS_NB
        default: return x;
    }
}
__device__ __forceinline__ double col_bcast(double x, int k) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = newbcast((unsigned)u, k), hi = newbcast((unsigned)(u >> 32), k);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// the value of lane 16 g + (lane % 16), g uniform: permlane16_swap of x with
// itself gives rows (0,0,2,2) and (1,1,3,3), permlane32_swap of one of those
// with itself its lower or upper half in both halves
__device__ __forceinline__ unsigned rowbcast(unsigned x, int g) {
    const auto q = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    const unsigned t = (g & 1) ? q[1] : q[0];
    const auto r = __builtin_amdgcn_permlane32_swap(t, t, false, false);
    return (g & 2) ? r[1] : r[0];
}
__device__ __forceinline__ double row_bcast(double x, int g) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = rowbcast((unsigned)u, g), hi = rowbcast((unsigned)(u >> 32), g);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// 1 / x: the hardware estimate refined by two Newton-Raphson steps
// (r <- r + r (1 - x r)), within an ulp or two of the quotient
__device__ __forceinline__ double recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

__device__ __forceinline__ double pick(const f64x4& t, int q) {
    return q == 0 ? t[0] : (q == 1 ? t[1] : (q == 2 ? t[2] : t[3]));
}

// the tile of X^T through the wave's LDS stage (exact; keeps the matrix cores
// free for products)
__device__ __forceinline__ f64x4 tr(const f64x4& x, double* st) {
    const int li = lane_i(), lk = lane_k();
#pragma unroll
    for (int v = 0; v < 4; ++v) st[(4 * v + lk) * 17 + li] = x[v];
    wave_sync_lds();
    f64x4 t;
#pragma unroll
    for (int v = 0; v < 4; ++v) t[v] = st[li * 17 + 4 * v + lk];
    wave_sync_lds();
    return t;
}
// (X + X^T) / 2 + add
__device__ __forceinline__ f64x4 symt(const f64x4& x, const f64x4& add, double* st) { return sym(x, tr(x, st), add); }

// ---------------------------------------------------------------------------
// Inverses by Gauss-Jordan elimination in the register layout.  The pivot's
// column reaches the lanes of each row of 16 by a DPP broadcast, the pivot row
// reaches the other rows of 16 by the permlane swaps.  Only the first n pivots
// are taken: the matrices are padded with the identity, on which the
// remaining steps change nothing.
// ---------------------------------------------------------------------------
// Symmetric positive definite a: the pivots are the diagonal, in order, and
// the inverse is formed in place.  `ok` is cleared by a pivot that is not
// positive (the matrix is not positive definite) or not finite.
// det (optional): the product of the pivots as a mantissa product and an
// exponent sum (the pivots are the diagonal of the LDL^T factorisation)
struct Det {
    double mant = 1.0;
    int exp = 0;
};
template <bool SPD = true>
__device__ __forceinline__ f64x4 inv_diag(f64x4 a, int n, bool& ok, Det* det = nullptr) {
    const int li = lane_i(), lk = lane_k();
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        if (k < n) {        // a guard, not an exit: the loop stays fully unrolled
            const int q = k >> 2, g = k & 3;
            const double pv = readlane_d(a[q], (g << 4) | k);          // a(k, k)
            double ck[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) ck[v] = col_bcast(a[v], k);    // a(4 v + lk, k)
            const double rk = row_bcast(a[q], g);                      // a(k, li)
            ok = ok && (SPD ? pv > 0.0 : pv != 0.0) && isfinite(pv);
            if (det) {
                int ex;
                det->mant *= frexp(pv, &ex);
                det->exp += ex;
            }
            const double r = recip(pv);
            const double rr = rk * r;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const double f = ck[v] * r;
                if (4 * v + lk == k) a[v] = li == k ? r : rr;           // the pivot row
                else a[v] = li == k ? -f : fma(-f, rk, a[v]);
            }
        }
    }
    return a;
}

__device__ __forceinline__ f64x4 inv_spd(const f64x4& a, int n, bool& ok) { return inv_diag<true>(a, n, ok); }

// General a: partial pivoting without row exchanges (the pivot of column k is
// the entry of largest magnitude among the rows not used yet, lower rows
// winning ties), elimination on [a | I]; row k of the inverse is then row p_k
// of the right half, gathered through the LDS stage.  `ok` is cleared by a
// zero or non-finite pivot.
__device__ __forceinline__ f64x4 inv_piv(f64x4 a, int n, double* st, bool& ok) {
    const int li = lane_i(), lk = lane_k();
    f64x4 b = eye();
    unsigned used = 0;
    unsigned long long perm = 0xFEDCBA9876543210ull;      // p_k = k beyond n
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        if (k >= n) continue;
        double ck[4];
        unsigned best = 0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            ck[v] = col_bcast(a[v], k);                          // a(4 v + lk, k)
            const int row = 4 * v + lk;
            // |entry| as float with the low mantissa bits dropped, then the row
            const unsigned bits = __float_as_uint((float)fabs(ck[v]));
            const unsigned key = ((used >> row) & 1u) ? 0u : (((bits >> 4) << 5) | 16u | (unsigned)(15 - row));
            best = best > key ? best : key;
        }
        const unsigned g0 = (unsigned)__builtin_amdgcn_readlane((int)best, 0);
        const unsigned g1 = (unsigned)__builtin_amdgcn_readlane((int)best, 16);
        const unsigned g2 = (unsigned)__builtin_amdgcn_readlane((int)best, 32);
        const unsigned g3 = (unsigned)__builtin_amdgcn_readlane((int)best, 48);
        const unsigned m01 = g0 > g1 ? g0 : g1, m23 = g2 > g3 ? g2 : g3;
        const unsigned key = m01 > m23 ? m01 : m23;
        const int p = 15 - (int)(key & 15u);
        used |= 1u << p;
        perm = (perm & ~(15ull << (4 * k))) | ((unsigned long long)p << (4 * k));
        const int q = p >> 2, g = p & 3;
        const double pv = readlane_d(pick(f64x4{ck[0], ck[1], ck[2], ck[3]}, q), g << 4);   // a(p, k)
        const double ra = row_bcast(pick(a, q), g);              // row p of a and of b
        const double rb = row_bcast(pick(b, q), g);
        ok = ok && pv != 0.0 && isfinite(pv);
        const double r = recip(pv);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const bool prow = 4 * v + lk == p;
            const double f = ck[v] * r;
            a[v] = prow ? ra * r : fma(-f, ra, a[v]);
            b[v] = prow ? rb * r : fma(-f, rb, b[v]);
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) st[(4 * v + lk) * 17 + li] = b[v];
    wave_sync_lds();
    f64x4 out;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int p = (int)((perm >> (4 * (4 * v + lk))) & 15ull);
        out[v] = st[p * 17 + li];
    }
    wave_sync_lds();
    return out;
}


__host__ __device__ inline int slices(int n) { return (n + 3) >> 2; }

// the identity beyond n on the diagonal of t
__device__ __forceinline__ f64x4 pad_eye(f64x4 t, int n) {
    const int li = lane_i(), lk = lane_k();
#pragma unroll
    for (int v = 0; v < 4; ++v)
        if (4 * v + lk == li && li >= n) t[v] = 1.0;
    return t;
}

}  // namespace w16
}  // namespace pks
