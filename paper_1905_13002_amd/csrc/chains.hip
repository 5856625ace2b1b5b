// chains.hip -- filter and smoother by overlapped chains (see chains.hpp).
//
// A wave runs four chains.  Every matrix of a chain, 4 x 4, is one double per
// lane (nx, ny <= 4, padded with zeros): lane j + 4 b + 16 i holds X(i, j) of
// chain b, the operand and result layout of v_mfma_f64_4x4x4_4b_f64, which
// multiplies four pairs of such tiles: mm(X, Y) = X^T Y.  Vectors are column 0.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "chains.hpp"
#include "tile16.hpp"

namespace pks {
namespace chains {

namespace {

constexpr int kAhead = 4;            // steps of a group; their loads are issued a group or two before
// Distances in the units of agree(), squared.  Two recursions of a CV model that
// have met stay within 2^-51 of each other (17000 samples): four times that is
// taken as having met.  Of an ill-conditioned model (a measurement much better than
// the prediction, or a badly conditioned S) they stay as far as 2^-45 apart, and no
// warm-up brings them closer: chains that differ by more than kSame are run again
// from their predecessor's end, a whole chain's length of steps further on, and
// then kRounding is enough where the first difference, `near`, says that what was
// not forgotten by then is by now (below 2^-50).
constexpr double kSame = 0x1p-98, kRounding = 0x1p-88;
// Means of settled models, 16 steps a product, have met at 2^-47.5; what they have not
// forgotten is below 2^-52 of where they started by the setup's count of steps
constexpr double kSameSettled = 0x1p-94;
constexpr double kTiny = 8.673617379884035e-19;       // 2^-60
constexpr double kMeet = 1e-11;      // how far a head's last covariance, formed step by step, may be from the doubled one
constexpr int kMaxLog = 9;           // settled after at most 2^kMaxLog steps
constexpr int kLongest = 384;        // and no later than this (a step of a head is 0.33 us of the filter, 0.5 of the smoother)

struct Lane {
    int j, b, i;
};
__device__ __forceinline__ Lane lane_of() {
    const int l = threadIdx.x & 63;
    return Lane{l & 3, (l >> 2) & 3, l >> 4};
}

__device__ __forceinline__ double mm(double x, double y, double acc = 0.0) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(x, y, acc, 0, 0, 0);
}
// X(i, P) in the lanes of row i
template <int P>
__device__ __forceinline__ double col(double x) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)u, 0x55 * P, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), 0x55 * P, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// X(P, j) in the lanes of column j: exact, a product with ones and zeros
template <int P>
__device__ __forceinline__ double row(double x, const Lane& t) { return mm(t.i == P ? 1.0 : 0.0, x); }
__device__ __forceinline__ double trans(double x, const Lane& t) { return mm(x, t.i == t.j ? 1.0 : 0.0); }
__device__ __forceinline__ double sym(double x, const Lane& t) { return 0.5 * (x + trans(x, t)); }

// the inverse of the symmetric 2 x 2 block at (P, P), zero elsewhere
template <int P>
__device__ __forceinline__ double inv2(double x, const Lane& t, bool& ok) {
    const double r0 = row<P>(x, t), r1 = row<P + 1>(x, t);
    const double a = col<P>(r0), b = col<P + 1>(r0), c = col<P + 1>(r1);
    const double det = fma(a, c, -b * b);
    ok &= (a > 0.0) & (det > 0.0);
    const double v = t.i != t.j ? -b : (t.i == P ? c : a);
    const bool in = (t.i >> 1) == P / 2 && (t.j >> 1) == P / 2;
    return in ? v * w16::recip(det) : 0.0;
}
// the inverse of a symmetric positive matrix: its leading N x N block, by 2 x 2
// blocks for N > 2 (an odd N has a one behind it)
template <int N>
__device__ __forceinline__ double inv(double x, const Lane& t, bool& ok) {
    if constexpr (N == 1) {
        const double a = col<0>(row<0>(x, t));
        ok &= a > 0.0;
        return t.i == 0 && t.j == 0 ? w16::recip(a) : 0.0;
    } else if constexpr (N == 2) {
        return inv2<0>(x, t, ok);
    } else {
        if (N == 3 && t.i == 3 && t.j == 3) x = 1.0;
        const double B = t.i < 2 && t.j > 1 ? x : 0.0, D = t.i > 1 && t.j > 1 ? x : 0.0;
        const double Ai = inv2<0>(x, t, ok);
        const double T = mm(Ai, B), TT = mm(B, Ai);            // A^-1 B and its transpose
        const double Si = inv2<2>(mm(-B, T, D), t, ok);
        const double U = mm(TT, Si), UT = mm(Si, TT);
        return mm(TT, UT, Ai + Si) - (U + UT);
    }
}
// whether its pivots are positive
template <int N>
__device__ __forceinline__ bool positive(double x, const Lane& t) {
    bool ok = true;
    if constexpr (N <= 2) {
        const double r0 = row<0>(x, t), a = col<0>(r0);
        ok = a > 0.0;
        if constexpr (N == 2) {
            const double b = col<1>(r0), c = col<1>(row<1>(x, t));
            ok &= fma(a, c, -b * b) > 0.0;
        }
    } else {
        (void)inv<N>(x, t, ok);
    }
    return ok;
}
// the inverse of a general N x N block, its pivots on the diagonal
template <int P>
__device__ __forceinline__ double pivot(double x, const Lane& t, bool& ok) {
    const double rp = row<P>(x, t), cp = col<P>(x), pv = col<P>(rp);
    ok &= fabs(pv) > 0.0;
    const double r = w16::recip(pv);
    const double rr = t.j == P ? r : rp * r;
    const double v = fma(-cp, rr, t.j == P ? 0.0 : x);
    return t.i == P ? rr : v;
}
template <int N>
__device__ __forceinline__ double inv_general(double x, const Lane& t, bool& ok) {
    x = pivot<0>(x, t, ok);
    if constexpr (N > 1) x = pivot<1>(x, t, ok);
    if constexpr (N > 2) x = pivot<2>(x, t, ok);
    if constexpr (N > 3) x = pivot<3>(x, t, ok);
    return x;
}
// x on all lanes of the lane's chain
__device__ __forceinline__ bool all_of(bool x, const Lane& t) {
    return (__ballot(!x) & (0x000f000f000f000full << (4 * t.b))) == 0;
}
// what a covariance P adds to C by way of A, A P A^T, is at most 2^-60 of C in
// every variance (A by its transpose)
__device__ __forceinline__ bool negligible(double AT, double P, double C, const Lane& t) {
    return all_of(t.i != t.j || mm(AT, mm(P, AT)) <= kTiny * C, t);
}

// ---------------------------------------------------------------------------
// where a lane finds its entries of a model's arrays
// ---------------------------------------------------------------------------
struct At {
    int ft, q, ht, r, v, w;                  // F^T, Q (and P), H^T, R, n-vectors, m-vectors
    bool nn, mn, mm, n, m;
};
__device__ __forceinline__ At at_of(const Lane& t, int nx, int ny) {
    At a;
    a.nn = t.i < nx && t.j < nx;
    a.mn = t.j < ny && t.i < nx;
    a.mm = t.i < ny && t.j < ny;
    a.n = t.j == 0 && t.i < nx;
    a.m = t.j == 0 && t.i < ny;
    a.ft = a.nn ? t.j * nx + t.i : 0;
    a.q = a.nn ? t.i * nx + t.j : 0;
    a.ht = a.mn ? t.j * nx + t.i : 0;
    a.r = a.mm ? t.i * ny + t.j : 0;
    a.v = a.n ? t.i : 0;
    a.w = a.m ? t.i : 0;
    return a;
}
__device__ __forceinline__ double pick(bool on, double x) { return on ? x : 0.0; }

// An array of one row of `words` T per step, from step k0 on: addressed by
// 32-bit offsets that advance with the groups, the steps of a group by a scalar
// one.  Entries outside (a lane without one, a step
// before or behind the array) read as zero and are not written.
constexpr unsigned kOutside = 0xc0000000u;             // a gigabyte from either end of an array's 2 GiB window
template <typename T>
struct Rows {
    __amdgpu_buffer_rsrc_t rs;
    unsigned at, step;                       // the lane's offset in the next group, bytes per step
    __device__ __forceinline__ void open(const T* p, int words, int64_t total, int64_t k0, int64_t k, bool on, int lane_at) {
        const int64_t left = p ? (total - k0) * words * (int64_t)sizeof(T) : 0;
        rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p) + (p ? k0 * words : 0), 0,
                                               (int)(left < 0x7fffffff ? left : 0x7fffffff), 0x00027000);
        step = words * (unsigned)sizeof(T);
        at = on ? (unsigned)((k - k0) * step) + lane_at * (unsigned)sizeof(T) : kOutside;
    }
    // (as it is stored: a conversion here would wait for the load)
    __device__ __forceinline__ T get(int s) const {
        if constexpr (sizeof(T) == 8)
            return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)at, (int)(s * step), 0));
        else
            return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)at, (int)(s * step), 0));
    }
    __device__ __forceinline__ void put(int s, double x, bool on) const {
        const int o = (int)(on ? at : kOutside), so = (int)(s * step);
        if constexpr (sizeof(T) == 8) {
            typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), rs, o, so, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, (float)x), rs, o, so, 0);
        }
    }
    __device__ __forceinline__ void move(int steps) { at += steps * step; }
};
__device__ __forceinline__ int64_t uniform(int64_t x) {
    return (int64_t)((uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)x) |
                     (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32);
}

struct Chain {
    int64_t c, b;                            // chain, sequence
    int64_t lo, hi;                          // the sequence's steps
    int64_t s, e;                            // the chain's own steps
    bool live;
};
__device__ __forceinline__ Chain chain_of(const Args& a, int64_t c) {
    Chain x;
    const int64_t n = a.offsets ? a.first[a.B] : (a.total + a.l - 1) / a.l;
    x.live = c < n;
    x.c = x.live ? c : n - 1;
    x.b = 0;
    x.lo = 0;
    x.hi = a.total;
    int64_t before = 0;
    if (a.offsets) {
        x.b = a.sequence[x.c];
        x.lo = a.offsets[x.b];
        x.hi = a.offsets[x.b + 1];
        before = a.first[x.b];
    }
    x.s = x.lo + (x.c - before) * a.l;
    x.e = min(x.s + a.l, x.hi);
    return x;
}

// P equals P2, each entry to kMeet of the root of the product of its variances
__device__ __forceinline__ bool meets(double P, double P2, const Lane& t) {
    const double D = t.i == t.j ? P2 : 0.0, di = mm(D, 1.0), dj = mm(1.0, D);
    return all_of((P - P2) * (P - P2) <= kMeet * kMeet * di * dj, t);
}
// moments (P, m) and (P2, m2) agree: differences against the standard deviations,
// the mean's against the size of the whole mean as well (its rounding is)
__device__ __forceinline__ bool agree(double P, double m, double P2, double m2, double far, const Lane& t) {
    const double D = t.i == t.j ? P2 : 0.0, di = mm(D, 1.0), dj = mm(1.0, D);
    const double zz = t.j == 0 && di > 0.0 ? m2 / sqrt(di) : 0.0;
    const double z = col<0>(row<0>(mm(zz, zz), t));
    const double dP = P - P2, dm = t.j == 0 ? m - m2 : 0.0;
    return all_of(dP * dP <= far * di * dj && dm * dm <= far * di * (1.0 + z), t);
}

// ---------------------------------------------------------------------------
// the steps
// ---------------------------------------------------------------------------
struct Row {
    double FT, Q, HT, R, u, y;               // y less d
};
template <int NY>
__device__ __forceinline__ void filter_step(const Row& x, const Lane& t, double& m, double& P, bool& ok) {
    // F P F^T + Q, symmetric in every bit: the two products are each other's
    // transposes.  (An antisymmetric part, once there, does not decay: without this two
    // recursions stay 2^-46 apart for good, with it they meet in every bit.)
    const double W = mm(P, x.FT), mp = mm(x.FT, m, x.u);
    const double Pp = 0.5 * (mm(x.FT, W, x.Q) + mm(W, x.FT, x.Q));
    const double V = mm(Pp, x.HT), VT = mm(x.HT, Pp);         // Pp H^T, H Pp
    const double Si = inv<NY>(mm(x.HT, V, x.R), t, ok);
    const double r = mm(x.HT, -mp, x.y);
    const double Z = mm(Si, VT);                              // K^T
    m = mm(Z, r, mp);
    P = mm(-VT, Z, Pp);
}
// the element's own factorisation (Lemma 1: H Q H^T + R), for its failure alone
template <int NY>
__device__ __forceinline__ bool row_ok(const Row& x, const Lane& t) {
    return positive<NY>(mm(x.HT, mm(x.Q, x.HT), x.R), t);
}
template <int NX>
__device__ __forceinline__ void smoother_gain(double FT, double Q, double u, double m, double P, const Lane& t, double& ET,
                                              double& Pp, double& mp, bool& ok) {
    const double FP = mm(FT, P);
    mp = mm(FT, m, u);
    Pp = mm(FT, mm(P, FT), Q);
    // (refined once: a product with an inverse alone loses the digits of Pp's condition)
    const double Pi = inv<NX>(Pp, t, ok), q = mm(Pi, FP);
    ET = mm(Pi, FP - mm(Pp, q), q);
}
__device__ __forceinline__ void smoother_step(double ET, double Pp, double mp, double m, double P, double& ms, double& Ps) {
    const double U = mm(Ps - Pp, ET);
    ms = mm(ET, ms - mp, m);
    Ps = mm(ET, U, P);
}

__device__ __forceinline__ void load_state(const double* p, int64_t c, const Lane& t, double& P, double& m) {
    P = p[c * kState + 4 * t.i + t.j];
    m = p[c * kState + 16 + 4 * t.i + t.j];
}
__device__ __forceinline__ void store_state(double* p, int64_t c, const Lane& t, double P, double m) {
    p[c * kState + 4 * t.i + t.j] = P;
    p[c * kState + 16 + 4 * t.i + t.j] = m;
}

// The second pass: whether a chain that entered with (P, m) runs again from its
// neighbour's end (P2, m2); one that does not keeps its own end
__device__ __forceinline__ bool again(const Args& a, const Chain& x, double P, double m, double P2, double m2, double met,
                                      double near, bool edge, const Lane& t) {
    const bool same = agree(P, m, P2, m2, met, t), close = agree(P, m, P2, m2, near, t);
    if (x.live && t.i == 0 && t.j == 0) a.forgets[x.c] = close;
    if (x.live && (same || edge)) {
        load_state(a.end[0], x.c, t, P, m);
        store_state(a.end[1], x.c, t, P, m);
    }
    return x.live && !same && !edge;
}
// The means of a settled model lose 30 bits in the steps that the covariances take
// to settle: what l steps bring below 2^-50
__device__ __forceinline__ double near_of(int64_t l, int head) {
    return exp2(2.0 * (fmin(30.0 * (double)l / head, 30.0) - 50.0));
}

// ---------------------------------------------------------------------------
// The flags, and the chains of every packed sequence.  A chain's wave reads its
// sequence from a table (a search would be ten loads in a row), which a wave a
// sequence fills: two sequences of 800 k steps with a model each, 209 us in all,
// 347 with a thread a sequence.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void set_flags(const Args& a) {
    if (a.reset || a.status[1] != kStatusMagic) {
        a.status[0] = kStatusOk;
        a.status[1] = kStatusMagic;
    }
    a.ctl[0] = 1;
}
__global__ __launch_bounds__(1024) void k_chain_setup(Args a) {
    __shared__ int64_t part[16], starts[1024];
    __shared__ int counts[1024];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (tid == 0) set_flags(a);
    int64_t before = 0;
    for (int b0 = 0; b0 < a.B; b0 += 1024) {
        const int b = b0 + tid;
        const int64_t own = b < a.B ? (a.offsets[b + 1] - a.offsets[b] + a.l - 1) / a.l : 0;
        int64_t inc = own;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t v = __shfl_up((long long)inc, d, 64);
            if (lane >= d) inc += v;
        }
        if (lane == 63) part[w] = inc;
        __syncthreads();
        int64_t ahead = before;
        for (int i = 0; i < 16; ++i) {
            if (i < w) ahead += part[i];
            before += part[i];
        }
        if (b < a.B) a.first[b] = ahead + inc - own;
        starts[tid] = ahead + inc - own;
        counts[tid] = (int)own;
        __syncthreads();
        const int n = min(1024, a.B - b0);
        for (int i = w; i < n; i += 16)              // a wave a sequence
            for (int c = lane; c < counts[i]; c += 64) a.sequence[starts[i] + c] = b0 + i;
        __syncthreads();
    }
    if (tid == 0) a.first[a.B] = before;
}

// ---------------------------------------------------------------------------
// Settled covariances of time-invariant models, four a wave: the filtering
// element of one step is doubled (Lemma 2 on equal elements) until each variance
// of A (P0 + C) A^T is at most 2^-60 of C's, after which every filtered covariance
// is C to FP64's rounding (see steady.hpp), and the smoothing element (Lemma 4)
// the same way; the powers then give the number of steps to 16.
// Bound by the latency of up to 2 kMaxLog dependent combines.
// ---------------------------------------------------------------------------
template <int NX, int NY>
__global__ __launch_bounds__(64) void k_chain_models(Args a) {
    const Lane t = lane_of();
    const int q = (int)blockIdx.x * 4 + t.b, b = q < a.B ? q : a.B - 1;
    const At at = at_of(t, a.nx, a.ny);
    const int64_t n2 = a.nx * a.nx, nm = a.nx * a.ny, m2 = a.ny * a.ny;
    const double FT = pick(at.nn, a.F[b * n2 + at.ft]), F = pick(at.nn, a.F[b * n2 + at.q]);
    const double Q = pick(at.nn, a.Q[b * n2 + at.q]), HT = pick(at.mn, a.H[b * nm + at.ht]);
    const double R = pick(at.mm, a.R[b * m2 + at.r]), P0 = pick(at.nn, a.P0[b * n2 + at.q]);
    const double u = a.u ? pick(at.n, a.u[(int64_t)b * a.nx + at.v]) : 0.0;
    const double d = a.d ? pick(at.m, a.d[(int64_t)b * a.ny + at.w]) : 0.0;
    const double I = t.i == t.j && t.i < a.nx ? 1.0 : 0.0;
    bool ok = true;
    double A, C, J;
    {
        const double QH = mm(Q, HT), HQ = mm(HT, Q), Si = inv<NY>(mm(HT, QH, R), t, ok);
        const double Kt = mm(Si, HQ), G = mm(HT, F);
        A = mm(-Kt, G, F);
        C = sym(mm(-Kt, HQ, Q), t);
        J = sym(mm(G, mm(Si, G)), t);
    }
    int lf = -1, le = -1;
    __shared__ double lev[kMaxLog][3][64];            // A, C, J of 2^l steps
    const int lane = threadIdx.x;
    auto combine = [&](double Ai, double Ci, double Aj, double Cj, double Jj, double& An, double& Cn, double& X, bool& fine) {
        const double M = mm(Ci, Jj, I);                       // I + C_i J_j
        X = inv_general<NX>(M, t, fine);
        // one Newton step, as the elimination has no row exchanges: leading minors of
        // I + C J may be small where it is not (correlated noise), and the step needs
        // a residual that is
        const double res = I - mm(trans(M, t), X);
        fine &= fabs(res) <= 1e-8;
        X = mm(trans(X, t), res, X);
        const double AX = mm(trans(Aj, t), X);                // A_j (I + C_i J_j)^-1
        An = mm(trans(AX, t), Ai);
        Cn = sym(mm(trans(mm(trans(AX, t), Ci), t), trans(Aj, t), Cj), t);
    };
    auto settled = [&](double An, double Cn) { return negligible(trans(An, t), P0 + Cn, Cn, t); };
    for (int l = 1; l <= kMaxLog; ++l) {
        lev[l - 1][0][lane] = A;
        lev[l - 1][1][lane] = C;
        lev[l - 1][2][lane] = J;
        bool fine = true;
        double An, Cn, X;
        combine(A, C, A, C, J, An, Cn, X, fine);
        const double JA = mm(J, A), Jn = sym(mm(JA, mm(trans(X, t), A), J), t);      // A^T J (I + C J)^-1 A + J
        const bool on = lf < 0, good = settled(An, Cn);
        ok &= fine || !on;
        A = on ? An : A;
        C = on ? Cn : C;
        J = on ? Jn : J;
        if (on && l >= 2 && good) lf = l;
        if (!__any(lf < 0)) break;
    }
    // the smallest multiple of 16 steps after which they have: 2^(lf - 1) have not
    int n16 = 16;
    {
        double Ac = 0.0, Cc = 0.0;
        for (int l = kMaxLog - 1; l >= 4; --l) {
            bool fine = true;
            double An, Cn, X;
            combine(Ac, Cc, lev[l][0][lane], lev[l][1][lane], lev[l][2][lane], An, Cn, X, fine);
            const bool done = settled(An, Cn) && all_of(fine, t), start = l == lf - 1, on = l < lf - 1 && !done;
            Ac = start ? lev[l][0][lane] : (on ? An : Ac);
            Cc = start ? lev[l][1][lane] : (on ? Cn : Cc);
            n16 += start || on ? 1 << l : 0;
        }
    }
    // settled gains
    const double P = C, W = mm(P, FT), Pp = sym(mm(FT, W, Q), t), VT = mm(HT, Pp);
    const double Kt = mm(inv<NY>(mm(HT, mm(Pp, HT), R), t, ok), VT);
    const double Phi = mm(-Kt, mm(HT, F), F), c = mm(-Kt, mm(HT, u, d), u);
    double ET, p2, m_;
    smoother_gain<NX>(FT, Q, 0.0, 0.0, P, t, ET, p2, m_, ok);
    double E2 = ET, L;
    {
        const double EFP = mm(ET, mm(FT, P));
        L = sym(P - EFP, t);
    }
    for (int l = 1; l <= kMaxLog; ++l) {
        lev[l - 1][0][lane] = E2;
        lev[l - 1][1][lane] = L;
        const double Ln = sym(mm(E2, mm(L, E2), L), t), En = mm(trans(E2, t), E2);     // (E E)^T
        const bool on = le < 0, good = negligible(En, P, Ln, t);
        L = on ? Ln : L;
        E2 = on ? En : E2;
        if (on && l >= 2 && good) le = l;
        if (!__any(le < 0)) break;
    }
    int e16 = 16;
    {
        double Ec = 0.0, Lc = 0.0;
        for (int l = kMaxLog - 1; l >= 4; --l) {
            const double El = lev[l][0][lane], Ll = lev[l][1][lane];
            const double Ln = sym(mm(Ec, mm(Ll, Ec), Lc), t), En = mm(trans(El, t), Ec);   // E_c L_l E_c^T + L_c, (E_c E_l)^T
            const bool fine = negligible(En, P, Ln, t), start = l == le - 1, on = l < le - 1 && !fine;
            Ec = start ? El : (on ? En : Ec);
            Lc = start ? Ll : (on ? Ln : Lc);
            e16 += start || on ? 1 << l : 0;
        }
    }
    const double PhiT = trans(Phi, t);
    if (q >= a.B) return;
    double* o = a.model + (int64_t)b * kModel + 4 * t.i + t.j;
    o[0] = PhiT;
    o[16] = Kt;
    o[32] = c;
    o[48] = P;
    o[64] = ET;
    o[80] = L;
    ok = ok && lf > 0 && le > 0;
    const bool good = all_of(ok, t) && n16 <= kLongest && e16 <= kLongest;
    if (t.i == 0 && t.j == 0) {
        if (!good) a.ctl[0] = 0;
        a.head[2 * b] = good ? n16 : 0;
        a.head[2 * b + 1] = good ? e16 : 0;
    }
}

// ---------------------------------------------------------------------------
// Whether a time-varying model forgets in time: the chains' passes are 0.33 us a
// step whether they are used or not.  kPilots waves follow at four places each what
// is left of a start (D, the product of the steps' (I - K H) F: a mean's error in
// standard deviations) for kPilotSteps steps, and note where the bits lost after half
// of them and all of them, carried on to the end of the second pass, are fewer than
// kNeed; two such notes end the attempt.  CV models, q / r from 40 to 0.0004 s^-3,
// carried on to 288 and 480 steps: within 5 bits of what is lost there up to 60 bits.
// 13 us before a pass of 265 (2^18 steps) to 470 (2^20); a model that does not
// forget: 2^18 steps 387 us, by the general scan alone 364, with the whole attempt
// before it 529.
// ---------------------------------------------------------------------------
constexpr int kPilots = 3, kPilotSteps = 48, kNote = 4;       // (notes: from word kNote of the flags)
constexpr double kNeed = 46.0;
__device__ __forceinline__ bool given_up(const Args& a) { return a.ctl[kNote] + a.ctl[kNote + 1] + a.ctl[kNote + 2] > 1; }

template <int NY>
__global__ __launch_bounds__(64) void k_chain_pilot(Args a) {
    if (blockIdx.x == kPilots) {                      // one sequence: the flags (k_chain_setup otherwise)
        if (threadIdx.x == 0) set_flags(a);
        return;
    }
    const Lane t = lane_of();
    const At at = at_of(t, a.nx, a.ny);
    const int64_t kb = a.total * (blockIdx.x + 1) / (kPilots + 1), k0 = kb + t.b * kPilotSteps;
    Rows<double> rFT, rQ, rHT, rR;
    rFT.open(a.F, a.nx * a.nx, a.total, kb, k0, at.nn, at.ft);
    rQ.open(a.Q, a.nx * a.nx, a.total, kb, k0, at.nn, at.q);
    rHT.open(a.H, a.nx * a.ny, a.total, kb, k0, at.mn, at.ht);
    rR.open(a.R, a.ny * a.ny, a.total, kb, k0, at.mm, at.r);
    Row cur[kAhead], nxt[kAhead];
    auto fetch = [&](Row (&r)[kAhead]) {
#pragma unroll
        for (int q = 0; q < kAhead; ++q) r[q] = Row{rFT.get(q), rQ.get(q), rHT.get(q), rR.get(q), 0.0, 0.0};
        rFT.move(kAhead);
        rQ.move(kAhead);
        rHT.move(kAhead);
        rR.move(kAhead);
    };
    double P = pick(at.nn, a.P0[at.q]), D = t.i == t.j ? sqrt(P) : 0.0;
    auto bits = [&] {
        const double di = mm(t.i == t.j ? P : 0.0, 1.0);
        double q = D != 0.0 ? D * D / di : 0.0;
#pragma unroll
        for (int s = 1; s < 64; s = s == 2 ? 16 : 2 * s) q = fmax(q, __shfl_xor(q, s, 64));
        return -0.5 * log2(q);
    };
    double half = 0.0;
    fetch(cur);
#pragma unroll 1
    for (int k = 0; k < kPilotSteps; k += kAhead) {
        if (k == kPilotSteps / 2) half = bits();
        fetch(nxt);
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            bool fine = true;
            filter_step<NY>(cur[q], t, D, P, fine);
            cur[q] = nxt[q];
        }
    }
    const double all = bits();
    const double lost = all + (all - half) * (double)(a.warm + a.l - kPilotSteps) / (kPilotSteps / 2);
    const unsigned long long few = __ballot(lost < kNeed && t.i == 0 && t.j == 0);
    if (threadIdx.x == 0) a.ctl[kNote + blockIdx.x] = __popcll(few) > 2;
}

// ---------------------------------------------------------------------------
// The chains.  Bound by the rows of the model (F, Q, H, R: 368 bytes a step at
// nx = 4, ny = 2 with y), which the warm-up reads again, and by the latency of a
// step (six dependent products and the inverse of S: 0.33 us): 4096 chains, a
// wave per SIMD, balance the two.  nx = 4, ny = 2, FP64, 2^20 steps: the filter
// 228 us, the smoother 220 us, where the block elements of the general
// scan took 464 us for the constants of every step and 760 us for the scans.
// ---------------------------------------------------------------------------
template <typename T, int NY>
__global__ __launch_bounds__(64) void k_chain_filter_tv(Args a, int pass) {
    if (pass ? a.ctl[0] == 0 : given_up(a)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) a.ctl[0] = 0;
        return;
    }
    const Lane t = lane_of();
    const Chain x = chain_of(a, (int64_t)blockIdx.x * 4 + t.b);
    const At at = at_of(t, a.nx, a.ny);
    const int n2 = a.nx * a.nx;
    const int64_t k0 = pass ? x.s : max(x.lo, x.s - a.warm);
    bool todo = x.live;
    double m, P;
    if (pass == 0) {
        const int64_t pr = a.each ? x.b : 0;
        P = pick(at.nn, a.P0[pr * n2 + at.q]);
        m = pick(at.n, a.m0[pr * a.nx + at.v]);
    } else {
        double oP, om;
        load_state(a.end[0], x.s > x.lo ? x.c - 1 : x.c, t, P, m);
        load_state(a.entry, x.c, t, oP, om);
        todo = again(a, x, oP, om, P, m, kSame, a.near, x.s == x.lo, t);
        if (!__any(todo)) return;
    }
    const int64_t kb = uniform(k0);                   // of the wave's first chain: the lowest
    int k = (int)(k0 - kb);
    const int s = (int)(x.s - kb), e = todo ? (int)(x.e - kb) : k;
    Rows<double> rFT, rQ, rHT, rR, ru, rd;
    Rows<T> ry, om, oP;
    rFT.open(a.F, n2, a.total, kb, k0, at.nn, at.ft);
    rQ.open(a.Q, n2, a.total, kb, k0, at.nn, at.q);
    rHT.open(a.H, a.nx * a.ny, a.total, kb, k0, at.mn, at.ht);
    rR.open(a.R, a.ny * a.ny, a.total, kb, k0, at.mm, at.r);
    ru.open(a.u, a.nx, a.total, kb, k0, at.n, at.v);
    rd.open(a.d, a.ny, a.total, kb, k0, at.m, at.w);
    ry.open(static_cast<const T*>(a.y), a.ny, a.total, kb, k0, at.m, at.w);
    om.open(static_cast<const T*>(a.m), a.nx, a.total, kb, k0, at.n, at.v);
    oP.open(static_cast<const T*>(a.P), n2, a.total, kb, k0, at.nn, at.q);
    bool ok = true;
    struct In {
        double FT, Q, HT, R, u, d;
        T y;
    } g[3][kAhead];
    auto fetch = [&](In (&r)[kAhead]) {
#pragma unroll
        for (int q = 0; q < kAhead; ++q)
            r[q] = In{rFT.get(q), rQ.get(q), rHT.get(q), rR.get(q), ru.get(q), rd.get(q), ry.get(q)};
        rFT.move(kAhead);
        rQ.move(kAhead);
        rHT.move(kAhead);
        rR.move(kAhead);
        ru.move(kAhead);
        rd.move(kAhead);
        ry.move(kAhead);
    };
    // straight-line code for a group: what does not depend on the moments fills the
    // latencies of what does.  Chains enter and end at a group's edge (the last
    // of a sequence aside, which nobody follows); steps beyond the end are dropped.
    auto use = [&](const In (&r)[kAhead]) {
        if (k == s && todo) store_state(a.entry, x.c, t, P, m);
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const bool out = k + q < e && k + q >= s;
            const Row z{r[q].FT, r[q].Q, r[q].HT, r[q].R, r[q].u, (double)r[q].y - r[q].d};
            bool fine = row_ok<NY>(z, t);
            filter_step<NY>(z, t, m, P, fine);
            ok &= fine | !out;
            oP.put(q, sym(P, t), out);
            om.put(q, m, out);
        }
        k += kAhead;
        om.move(kAhead);
        oP.move(kAhead);
        if (k == e && todo) store_state(a.end[pass], x.c, t, P, m);
    };
    fetch(g[0]);
    fetch(g[1]);
    while (__any(k < e)) {
        fetch(g[2]);
        use(g[0]);
        fetch(g[0]);
        use(g[1]);
        fetch(g[1]);
        use(g[2]);
    }
    if (!ok) a.ctl[0] = 0;
}

template <typename T, int NX>
__global__ __launch_bounds__(64) void k_chain_smoother_tv(Args a, int pass) {
    if (a.ctl[0] == 0) return;
    const Lane t = lane_of();
    const Chain x = chain_of(a, (int64_t)blockIdx.x * 4 + t.b);
    const At at = at_of(t, a.nx, a.ny);
    const int n2 = a.nx * a.nx;
    const int64_t from = pass ? x.e : min(x.e - 1 + a.warm, x.hi - 1);      // the step with known moments
    const int64_t kb = uniform(x.s);                  // of the wave's first chain: the lowest step
    bool todo = x.live;
    double ms, Ps;
    if (pass == 0) {
        Ps = pick(at.nn, (double)static_cast<const T*>(a.P)[from * n2 + at.q]);
        ms = pick(at.n, (double)static_cast<const T*>(a.m)[from * a.nx + at.v]);
        if (x.live && from < x.e) {                   // a sequence's last step
            if (at.nn) static_cast<T*>(a.Ps)[from * n2 + at.q] = (T)Ps;
            if (at.n) static_cast<T*>(a.ms)[from * a.nx + at.v] = (T)ms;
        }
    } else {
        double oP, om;
        load_state(a.end[0], x.e < x.hi ? x.c + 1 : x.c, t, Ps, ms);
        load_state(a.entry, x.c, t, oP, om);
        todo = again(a, x, oP, om, Ps, ms, kSame, a.near, x.e == x.hi, t);
        if (!__any(todo)) return;
    }
    // groups of kAhead steps that end at s exactly: rows below it are never formed
    const int s = (int)(x.s - kb), e = (int)(x.e - kb), top = (int)(from - kb);
    int k = todo ? s + (top - s + kAhead - 1) / kAhead * kAhead - kAhead : s - kAhead;       // a group's lowest step
    const int64_t kl = kb + k;
    Rows<double> rFT, rQ, ru;
    Rows<T> rm, rP, om, oP;
    rFT.open(a.F, n2, a.total, kb + 1, kl + 1, at.nn, at.ft);       // out of a step: the next one's rows
    rQ.open(a.Q, n2, a.total, kb + 1, kl + 1, at.nn, at.q);
    ru.open(a.u, a.nx, a.total, kb + 1, kl + 1, at.n, at.v);
    rm.open(static_cast<const T*>(a.m), a.nx, a.total, kb, kl, at.n, at.v);
    rP.open(static_cast<const T*>(a.P), n2, a.total, kb, kl, at.nn, at.q);
    om.open(static_cast<const T*>(a.ms), a.nx, a.total, kb, kl, at.n, at.v);
    oP.open(static_cast<const T*>(a.Ps), n2, a.total, kb, kl, at.nn, at.q);
    bool ok = true;
    struct In {
        double FT, Q, u;
        T m, P;
    } g[3][kAhead];
    auto fetch = [&](In (&r)[kAhead]) {
#pragma unroll
        for (int q = 0; q < kAhead; ++q) r[q] = In{rFT.get(q), rQ.get(q), ru.get(q), rm.get(q), rP.get(q)};
        rFT.move(-kAhead);
        rQ.move(-kAhead);
        ru.move(-kAhead);
        rm.move(-kAhead);
        rP.move(-kAhead);
    };
    auto use = [&](const In (&r)[kAhead]) {
        if (k + kAhead == e && todo) store_state(a.entry, x.c, t, Ps, ms);
#pragma unroll
        for (int q = kAhead - 1; q >= 0; --q) {
            double ET, Pp, mp;
            bool fine = true;
            const double m = (double)r[q].m, P = (double)r[q].P;
            smoother_gain<NX>(r[q].FT, r[q].Q, r[q].u, m, P, t, ET, Pp, mp, fine);
            const bool on = k + q < top, out = k + q < e && k >= s;
            double mn = ms, Pn = Ps;
            smoother_step(ET, Pp, mp, m, P, mn, Pn);
            ms = on ? mn : ms;
            Ps = on ? Pn : Ps;
            ok &= fine | !(out && on);
            oP.put(q, sym(Ps, t), out && on);
            om.put(q, ms, out && on);
        }
        if (k == s && todo) store_state(a.end[pass], x.c, t, Ps, ms);
        k -= kAhead;
        om.move(-kAhead);
        oP.move(-kAhead);
    };
    if (todo && k < s) store_state(a.end[pass], x.c, t, Ps, ms);       // a chain of one step, the sequence's last
    fetch(g[0]);
    fetch(g[1]);
    while (__any(k >= s)) {
        fetch(g[2]);
        use(g[0]);
        fetch(g[0]);
        use(g[1]);
        fetch(g[1]);
        use(g[2]);
    }
    if (!ok) a.ctl[0] = 0;
}

// ---------------------------------------------------------------------------
// Time-invariant models, one per sequence.  Beyond a sequence's first `head`
// steps (and before its last, for the smoother) the covariances and gains are
// the settled ones, and what is left of a step is m_k = A m_{k-1} + B z_k + c
// (filter: A = Phi, B = K, z = y; smoother, backwards: A = E, B = I - E F, z the
// filtered mean).  16 steps at a time, z_{4 j + q} as column j of tile q:
//   S      the mean before steps 0, 4, 8, 12: a chain of four products with A^4,
//          from the columns' inputs A^3 B z_0 + A^2 B z_1 + A B z_2 + B z_3 + c';
//   O_q    the means of steps q, 4 + q, 8 + q, 12 + q, O_q = A O_{q-1} + B Z_q + c.
// 14 products for 16 steps, 8 where only the last is wanted.
// Chains that start in there run the means alone from 1 3/4 times the steps that
// the covariances take to settle (the mean forgets at half their rate, and they
// settle 2^-60 deep: 2^-52); those whose start would fall into the head start
// with the sequence.
// Bound by the slowest head (0.33 us a step of the filter, and as the smoother's
// tail and head 0.2 and 0.45) beside the rows to write: 8.5 M steps of 1024 CV
// models, mixed: filter 193 us, smoother 323; the general scan, 1225 in all.  Loads
// are eight groups ahead, and
// results are written a row a lane: in pieces of 16 bytes the filter took 30 us
// more.
// ---------------------------------------------------------------------------
constexpr int kLong = 16;            // steps of a group
constexpr int kPace = 4;             // stores in flight of a wave that writes settled rows
constexpr int kWriters = 512;        // of such waves
constexpr int kDeep = 8;             // groups whose loads are in flight

__device__ __forceinline__ double pick_of(int j, double a, double b, double c, double d) {
    const double lo = j & 1 ? b : a, hi = j & 1 ? d : c;
    return j & 2 ? hi : lo;
}

struct Affine {
    double AT, A4T, BT, c;                   // tiles of A^T, (A^4)^T, B^T; c in all columns
    double BqT[4], c4;                       // of A^{3-q} B; the constant of four steps
    __device__ __forceinline__ void set(double at, double bt, double c0, const Lane& t) {
        AT = at;
        BT = bt;
        c = c0;
        const double A = trans(at, t);
        // (X Y)^T = mm(Y, X^T)
        const double A2T = mm(A, AT);
        A4T = mm(trans(A2T, t), A2T);
        BqT[3] = bt;
        c4 = c0;
#pragma unroll
        for (int q = 2; q >= 0; --q) {
            BqT[q] = mm(trans(BqT[q + 1], t), AT);
            c4 = mm(AT, c4, c0);
        }
    }
    // m: the mean before the group (in every column), then the one after it; BACK:
    // the steps from the last to the first, tiles and columns in reverse
    template <bool BACK>
    __device__ __forceinline__ void run(double& m, const double (&z)[4], double (&o)[4], bool rows, const Lane& t) const {
        double in = c4;
#pragma unroll
        for (int q = 0; q < 4; ++q) in = mm(BqT[q], z[BACK ? 3 - q : q], in);
        const double s0 = m, s1 = mm(A4T, s0, col<BACK ? 3 : 0>(in)), s2 = mm(A4T, s1, col<BACK ? 2 : 1>(in)),
                     s3 = mm(A4T, s2, col<BACK ? 1 : 2>(in));
        m = mm(A4T, s3, col<BACK ? 0 : 3>(in));
        if (!rows) return;
        const int j = BACK ? 3 - t.j : t.j;
        double x = pick_of(j, s0, s1, s2, s3);
#pragma unroll
        for (int q = 0; q < 3; ++q) o[BACK ? 3 - q : q] = x = mm(AT, x, mm(BT, z[BACK ? 3 - q : q], c));
        o[BACK ? 0 : 3] = pick_of(j, s1, s2, s3, m);
    }
};

// column j of the lane's row -> column j - 1 (and 0 -> 3), or the other way
template <bool UP>
__device__ __forceinline__ double turn(double x) {
    constexpr int ctl = UP ? (3 | 0 << 2 | 1 << 4 | 2 << 6) : (1 | 2 << 2 | 3 << 4 | 0 << 6);
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)u, ctl, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), ctl, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// vectors of 16 rows: tile q has row 4 j + q as column j
template <typename T>
__device__ __forceinline__ void open_cols(Rows<T>& r, const T* p, int words, int64_t total, int64_t k0, int64_t k,
                                          const Lane& t) {
    r.open(p, words, total, k0, k, t.i < words, 4 * t.j * words + t.i);
}
// end of the steps with settled covariances that start at lo + head
__device__ __forceinline__ int64_t settled_end(int64_t lo, int64_t hi, int tail, bool smoothed) {
    return smoothed ? lo + ((hi - lo - tail) & -(int64_t)kLong) : hi;
}
// The settled covariance in all the rows that hold it: a wave's share is a
// contiguous range of rows, written 16 bytes a lane (NX = 4).  Waves of their own,
// behind the chains' in the same launch, each with few stores in flight: the
// chains' loads and stores queue behind them.  8.5 M steps, FP32, 100 us by
// themselves; beside the chains they add 165 us if those write them, 100 with
// stores unpaced, 47 with four in flight.
template <typename T, int NX, bool SMOOTHED>
__device__ __forceinline__ void write_settled(const Args& a, int64_t w, int64_t nw, T* dst) {
    typedef unsigned unit_t __attribute__((ext_vector_type(NX == 4 ? 4 : sizeof(T) / 4)));
    constexpr int n2 = NX * NX, V = sizeof(unit_t) / sizeof(T), U = n2 / V, L = 64 / U * U;     // units a row, lanes in use
    const int lane = threadIdx.x & 63, part = lane % U;
    int64_t r = a.total * w / nw;
    const int64_t r1 = a.total * (w + 1) / nw;
    if (r >= r1 || lane >= L) return;
    int lo = 0, hi = a.B;                             // offsets[lo] <= r < offsets[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (a.offsets[mid] <= r) lo = mid; else hi = mid;
    }
    for (int b = lo; r < r1; ++b) {
        const int64_t s = a.offsets[b], e = a.offsets[b + 1];
        const int head = a.head[2 * b], tail = a.head[2 * b + 1];
        const int64_t c0 = max(r, s + head), c1 = min(r1, settled_end(s, e, tail, SMOOTHED));
        if (c0 < c1) {
            T v[V];
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const int q = part * V + i;
                v[i] = (T)a.model[(int64_t)b * kModel + (SMOOTHED ? 80 : 48) + q / NX * 4 + q % NX];
            }
            unit_t x;
            __builtin_memcpy(&x, v, sizeof x);
            unit_t* p = reinterpret_cast<unit_t*>(dst + c0 * n2) + lane;
            const int64_t units = (c1 - c0) * U;
            int64_t q = lane;
            for (; q + (kPace / 2 - 1) * L < units; q += kPace / 2 * L) {
#pragma unroll
                for (int i = 0; i < kPace / 2; ++i, p += L) __builtin_memcpy(p, &x, sizeof x);
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kPace / 2) : "memory");
            }
            for (; q < units; q += L, p += L) __builtin_memcpy(p, &x, sizeof x);
        }
        r = min(e, r1);
    }
}

// the vectors of 16 steps, o_q(i, j) entry i of step 4 j + q: written a row a
// lane by way of LDS (NX = 4; else as they lie): 256 or 512 consecutive bytes a
// chain and store, not 16 pieces
template <typename T, int NX>
struct OutRows {
    Rows<T> r;
    T* st;
    __device__ __forceinline__ void open(const T* p, int64_t total, int64_t k0, int64_t k, const Lane& t, T* lds) {
        if constexpr (NX == 4) {
            r.open(p, NX, total, k0, k, true, NX * (4 * t.i + t.j));
            st = lds + 64 * t.b;
        } else {
            open_cols(r, p, NX, total, k0, k, t);
        }
    }
    // the rows k .. end - 1 of the group
    __device__ __forceinline__ void put(const double (&o)[4], int k, int end, const Lane& t) const {
        if constexpr (NX == 4) {
            typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
            for (int q = 0; q < 4; ++q) st[(4 * t.j + q) * 4 + t.i] = (T)o[q];
            w16::wave_sync_lds();
            const int at = (int)(k + 4 * t.i + t.j < end ? r.at : kOutside);
#pragma unroll
            for (int h = 0; h < (int)sizeof(T) / 4; ++h) {
                u32x4 x;
                __builtin_memcpy(&x, reinterpret_cast<const char*>(st + (4 * t.i + t.j) * 4) + 16 * h, 16);
                __builtin_amdgcn_raw_buffer_store_b128(x, r.rs, at, 16 * h, 0);
            }
            w16::wave_sync_lds();
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) r.put(q, o[q], k + 4 * t.j + q < end);
        }
    }
};

template <typename T, int NX, int NY>
__global__ __launch_bounds__(64) void k_chain_filter_ti(Args a, int pass, int writers) {
    __shared__ __align__(16) T stage[256];
    if (a.ctl[0] == 0) return;
    const int chains = gridDim.x - writers;           // waves of chains, then of settled rows
    if ((int)blockIdx.x >= chains)
        return write_settled<T, NX, false>(a, blockIdx.x - chains, writers, static_cast<T*>(a.P));
    const Lane t = lane_of();
    const Chain x = chain_of(a, (int64_t)blockIdx.x * 4 + t.b);
    const At at = at_of(t, NX, NY);
    constexpr int n2 = NX * NX;
    const double* md = a.model + x.b * kModel + 4 * t.i + t.j;
    const double Pstar = md[48];
    const int head = a.head[2 * x.b];
    const int64_t warm = (head + head / 2 + head / 4 + kLong - 1) & -kLong;
    int64_t k0 = pass ? x.s : x.s - warm;
    if (pass == 0 && k0 < x.lo + head) k0 = x.lo;
    bool todo = x.live;
    double m, P;
    if (pass == 0) {
        P = k0 == x.lo ? pick(at.nn, a.P0[x.b * n2 + at.q]) : Pstar;
        m = t.i < NX ? a.m0[x.b * NX + (t.i < NX ? t.i : 0)] : 0.0;
    } else {
        double oP, om;
        load_state(a.end[0], x.s > x.lo ? x.c - 1 : x.c, t, P, m);
        load_state(a.entry, x.c, t, oP, om);
        todo = again(a, x, oP, om, P, m, kSameSettled, near_of(a.l, head), x.s == x.lo, t);
        if (!__any(todo)) return;
    }
    const double FT = pick(at.nn, a.F[x.b * n2 + at.ft]), Q = pick(at.nn, a.Q[x.b * n2 + at.q]);
    const double HT = pick(at.mn, a.H[x.b * (NX * NY) + at.ht]), R = pick(at.mm, a.R[x.b * (NY * NY) + at.r]);
    const double u = a.u && t.i < NX ? a.u[x.b * NX + t.i] : 0.0, d = a.d && t.i < NY ? a.d[x.b * NY + t.i] : 0.0;
    Affine f;
    f.set(md[0], md[16], col<0>(md[32]), t);
    // chains of a wave need not start in order: the lowest start is the base
    int64_t kb = k0;
#pragma unroll
    for (int s = 4; s < 16; s <<= 1) kb = min(kb, (int64_t)__shfl_xor((long long)kb, s, 64));
    kb = uniform(kb);
    int k = (int)(k0 - kb);
    const int s = (int)(x.s - kb), e = todo ? (int)(x.e - kb) : k, settled = (int)(x.lo + head - kb);
    Rows<T> ry, oP;
    open_cols(ry, static_cast<const T*>(a.y), NY, a.total, kb, k0, t);
    OutRows<T, NX> om;
    om.open(static_cast<const T*>(a.m), a.total, kb, k0, t, stage);
    oP.open(static_cast<const T*>(a.P), n2, a.total, kb, k0, at.nn, at.q);
    bool ok = true;
    auto fetch = [&](T (&r)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) r[q] = ry.get(q);
        ry.move(kLong);
    };
    auto begin = [&] {
        if (k == s && todo) store_state(a.entry, x.c, t, P, m);
    };
    auto finish = [&](const double (&o)[4]) {
        if (__any(k >= s && k < e)) om.put(o, k, k >= s ? e : k, t);
        k += kLong;
        om.r.move(kLong);
        if (k == e && todo) store_state(a.end[pass], x.c, t, P, m);
    };
    // heads of sequences: the first groups of chains that start with one
    if (__any(k < settled && k < e)) {
        T cur[4], nxt[4];
        fetch(cur);
        while (__any(k < settled && k < e)) {
            fetch(nxt);
            begin();
            double z[4] = {(double)cur[0], (double)cur[1], (double)cur[2], (double)cur[3]}, o[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    bool fine = true;
                    filter_step<NY>(Row{FT, Q, HT, R, u, col<0>(z[q]) - d}, t, m, P, fine);
                    P = k >= settled ? Pstar : P;
                    o[q] = t.j == j ? m : o[q];
                    const bool put = k >= s && k + 4 * j + q < e;
                    ok &= fine | !put;
                    oP.put(q, sym(P, t), put && k < settled);
                    z[q] = turn<false>(z[q]);
                }
                oP.move(4);
            }
            finish(o);
            if (__any(k == settled && k <= e)) {
                const bool same = meets(P, Pstar, t);
                ok &= same | !(k == settled && k <= e);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) cur[q] = nxt[q];
        }
        ry.move(-kLong);
    }
    P = Pstar;
    T g[kDeep][4];
#pragma unroll
    for (int i = 0; i < kDeep; ++i) fetch(g[i]);
    while (__any(k < e)) {
#pragma unroll
        for (int i = 0; i < kDeep; ++i) {
            const double y[4] = {(double)g[i][0], (double)g[i][1], (double)g[i][2], (double)g[i][3]};
            double o[4] = {0.0, 0.0, 0.0, 0.0};
            begin();
            f.template run<false>(m, y, o, __any(k >= s && k < e), t);
            finish(o);
            fetch(g[i]);
        }
    }
    if (!ok) a.ctl[0] = 0;
}

template <typename T, int NX>
__global__ __launch_bounds__(64) void k_chain_smoother_ti(Args a, int pass, int writers) {
    __shared__ __align__(16) T stage[256];
    if (a.ctl[0] == 0) return;
    const int chains = gridDim.x - writers;
    if ((int)blockIdx.x >= chains)
        return write_settled<T, NX, true>(a, blockIdx.x - chains, writers, static_cast<T*>(a.Ps));
    const Lane t = lane_of();
    const Chain x = chain_of(a, (int64_t)blockIdx.x * 4 + t.b);
    const At at = at_of(t, NX, 1);
    constexpr int n2 = NX * NX;
    const double* md = a.model + x.b * kModel + 4 * t.i + t.j;
    const double Pstar = md[48], ETs = md[64], Psstar = md[80];
    const int head = a.head[2 * x.b], tail = a.head[2 * x.b + 1];
    const int64_t warm = (tail + tail / 2 + tail / 4 + kLong - 1) & -kLong;
    int64_t from = pass ? x.e : x.e + warm;          // the step with known moments
    if (from > x.hi - 1 - tail && (pass == 0 || x.e == x.hi)) from = x.hi - 1;
    bool todo = x.live;
    double ms, Ps;
    if (pass == 0) {
        const double Pl = pick(at.nn, (double)static_cast<const T*>(a.P)[from * n2 + at.q]);
        ms = t.i < NX ? (double)static_cast<const T*>(a.m)[from * NX + t.i] : 0.0;
        const double Pend = x.hi - x.lo >= head ? Pstar : Pl;
        Ps = from < x.hi - 1 ? Psstar : Pend;
        if (x.live && from < x.e) {                   // a sequence's last step
            if (at.nn) static_cast<T*>(a.Ps)[from * n2 + at.q] = (T)Pend;
            if (at.n) static_cast<T*>(a.ms)[from * NX + at.v] = (T)ms;
        }
    } else {
        double oP, om;
        load_state(a.end[0], x.e < x.hi ? x.c + 1 : x.c, t, Ps, ms);
        load_state(a.entry, x.c, t, oP, om);
        todo = again(a, x, oP, om, Ps, ms, kSameSettled, near_of(a.l, tail), x.e == x.hi, t);
        if (!__any(todo)) return;
    }
    const double FT = pick(at.nn, a.F[x.b * n2 + at.ft]), Q = pick(at.nn, a.Q[x.b * n2 + at.q]);
    const double u = a.u && t.i < NX ? a.u[x.b * NX + t.i] : 0.0;
    const double Pps = mm(FT, mm(Pstar, FT), Q);      // F P F^T + Q, settled
    Affine f;
    {
        // B = I - E F, c = -E u
        const double I = t.i == t.j && t.i < NX ? 1.0 : 0.0;
        f.set(ETs, trans(I - mm(ETs, trans(FT, t)), t), -mm(ETs, u), t);
    }
    const int64_t kb = uniform(x.s);                  // of the wave's first chain: the lowest step
    const int s = (int)(x.s - kb), e = (int)(x.e - kb), top = (int)(from - kb);
    const int first = (int)(x.lo + head - 1 - kb);    // P has settled from here on
    const int last = (int)(x.hi - 1 - tail - kb);     // Ps has up to here
    int k = todo ? s + (top - s + kLong - 1) / kLong * kLong - kLong : s - kLong;       // a group's lowest step
    const int64_t kl = kb + k;
    Rows<T> rm, rP, oP;
    open_cols(rm, static_cast<const T*>(a.m), NX, a.total, kb, kl, t);
    rP.open(static_cast<const T*>(a.P), n2, a.total, kb, kl, at.nn, at.q);
    OutRows<T, NX> om;
    om.open(static_cast<const T*>(a.ms), a.total, kb, kl, t, stage);
    oP.open(static_cast<const T*>(a.Ps), n2, a.total, kb, kl, at.nn, at.q);
    bool ok = true;
    auto fetch = [&](T (&r)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) r[q] = rm.get(q);
        rm.move(-kLong);
    };
    auto begin = [&] {
        if (k + kLong == e && todo) store_state(a.entry, x.c, t, Ps, ms);
    };
    auto finish = [&](const double (&o)[4]) {
        const int end = k >= s ? min(e, top) : k;     // rows to write: k .. end - 1
        if (__any(k < end)) om.put(o, k, end, t);
        if (k == s && todo) store_state(a.end[pass], x.c, t, Ps, ms);
        k -= kLong;
        om.r.move(-kLong);
    };
    // the chain's group has rows of the sequence's head or tail
    auto edge = [&](int kk) { return kk >= s && (kk < first || kk + kLong - 1 > last); };
    if (todo && k < s) store_state(a.end[pass], x.c, t, Ps, ms);       // a chain of one step, the sequence's last
    int at_k = k;                                     // where rP and oP stand
    while (__any(k >= s)) {
        if (__any(edge(k))) {
            rP.move(k - at_k);
            oP.move(k - at_k);
            T cur[4], nxt[4], Pc[kLong], Pn[kLong];
            auto fetch_P = [&](T (&r)[kLong], int kk) {       // of the head, all else is known
                if (__any(kk >= s && kk < first)) {
#pragma unroll
                    for (int q = 0; q < kLong; ++q) r[q] = rP.get(q);
                } else {
#pragma unroll
                    for (int q = 0; q < kLong; ++q) r[q] = T(0);
                }
                rP.move(-kLong);
            };
            fetch(cur);
            fetch_P(Pc, k);
            while (__any(edge(k))) {
                fetch(nxt);
                fetch_P(Pn, k - kLong);
                begin();
                const int end = k >= s ? min(e, top) : k;
                const bool mine = edge(k);
                const bool varies = __any(k >= s && k < first);
                double z[4] = {(double)cur[0], (double)cur[1], (double)cur[2], (double)cur[3]}, o[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int j = 3; j >= 0; --j) {
                    double ET[4], Pp[4], mp[4], mq[4], P[4];
#pragma unroll
                    for (int q = 3; q >= 0; --q) {
                        mq[q] = col<3>(z[q]);
                        z[q] = turn<true>(z[q]);
                        P[q] = k + 4 * j + q >= first ? Pstar : (double)Pc[4 * j + q];
                    }
                    if (varies) {                     // four gains, independent of each other
#pragma unroll
                        for (int q = 3; q >= 0; --q) {
                            bool fine = true;
                            smoother_gain<NX>(FT, Q, u, mq[q], P[q], t, ET[q], Pp[q], mp[q], fine);
                            ok &= fine | !(k + 4 * j + q < end);
                        }
                    } else {
#pragma unroll
                        for (int q = 3; q >= 0; --q) {
                            ET[q] = ETs;
                            Pp[q] = Pps;
                            mp[q] = mm(FT, mq[q], u);
                        }
                    }
#pragma unroll
                    for (int q = 3; q >= 0; --q) {
                        const int kq = k + 4 * j + q;
                        const bool on = kq < top;
                        double mn = ms, Psn = Ps;
                        smoother_step(ET[q], Pp[q], mp[q], mq[q], P[q], mn, Psn);
                        ms = on ? mn : ms;
                        const bool enters = on && kq == last && kq >= first && k >= s;
                        if (__any(enters)) {
                            const bool same = meets(Psn, Psstar, t);
                            ok &= same | !enters;
                        }
                        Ps = on ? (kq >= first && kq <= last ? Psstar : Psn) : Ps;
                        o[q] = t.j == j ? ms : o[q];
                        oP.put(4 * j + q, sym(Ps, t), kq < end && mine);
                    }
                }
                oP.move(-kLong);
                finish(o);
#pragma unroll
                for (int q = 0; q < 4; ++q) cur[q] = nxt[q];
#pragma unroll
                for (int q = 0; q < kLong; ++q) Pc[q] = Pn[q];
            }
            rm.move(kLong);                           // (one group was fetched ahead)
            rP.move(kLong);
            at_k = k;
        } else {
            Ps = Psstar;
            T g[kDeep][4];
#pragma unroll
            for (int i = 0; i < kDeep; ++i) fetch(g[i]);
            bool more = true;
            while (more) {
#pragma unroll
                for (int i = 0; i < kDeep; ++i) {
                    const double m[4] = {(double)g[i][0], (double)g[i][1], (double)g[i][2], (double)g[i][3]};
                    double o[4] = {0.0, 0.0, 0.0, 0.0};
                    begin();
                    f.template run<true>(ms, m, o, __any(k >= s && k < min(e, top)), t);
                    finish(o);
                    if (!__any(k >= s) || __any(edge(k))) {
                        more = false;
                        break;
                    }
                    fetch(g[i]);
                }
            }
            // back to the group after the last one taken
            rm.move(kLong * kDeep - kLong);
        }
    }
    if (!ok) a.ctl[0] = 0;
}

// ---------------------------------------------------------------------------
// a chain that still did not enter with its neighbour's end clears the flag
// ---------------------------------------------------------------------------
template <bool SMOOTHER>
__global__ __launch_bounds__(64) void k_chain_check(Args a) {
    if (a.ctl[0] == 0) return;
    const Lane t = lane_of();
    const Chain x = chain_of(a, (int64_t)blockIdx.x * 4 + t.b);
    const bool edge = SMOOTHER ? x.e == x.hi : x.s == x.lo;
    double P, m, P2, m2;
    load_state(a.entry, x.c, t, P, m);
    load_state(a.end[1], edge ? x.c : (SMOOTHER ? x.c + 1 : x.c - 1), t, P2, m2);
    const bool same = agree(P, m, P2, m2, kSame, t), close = agree(P, m, P2, m2, kRounding, t);
    if (x.live && !edge && !same && !(close && a.forgets[x.c])) a.ctl[0] = 0;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
template <typename F>
void timed(const char* name, hipStream_t s, F&& f) {
    prof_begin(name, s);
    f();
    prof_end(s);
}

template <typename T, int NX, int NY>
hipError_t run(const Args& a, bool tv, hipStream_t s) {
    const int writers = kWriters;
    const dim3 grid((unsigned)((a.max_chains + 3) / 4)), more(grid.x + writers), wave(64);
    if (a.offsets) timed("k_chain_setup", s, [&] { hipLaunchKernelGGL(k_chain_setup, dim3(1), dim3(1024), 0, s, a); });
    if (tv)
        timed("k_chain_pilot", s,
              [&] { hipLaunchKernelGGL((k_chain_pilot<NY>), dim3(kPilots + (a.offsets ? 0 : 1)), wave, 0, s, a); });
    else
        timed("k_chain_models", s,
              [&] { hipLaunchKernelGGL((k_chain_models<NX, NY>), dim3((a.B + 3) / 4), wave, 0, s, a); });
    for (int pass = 0; pass < 2; ++pass)
        timed(pass ? "k_chain_filter_again" : "k_chain_filter", s, [&] {
            if (tv) hipLaunchKernelGGL((k_chain_filter_tv<T, NY>), grid, wave, 0, s, a, pass);
            else hipLaunchKernelGGL((k_chain_filter_ti<T, NX, NY>), pass ? grid : more, wave, 0, s, a, pass, pass ? 0 : writers);
        });
    timed("k_chain_check", s, [&] { hipLaunchKernelGGL((k_chain_check<false>), grid, wave, 0, s, a); });
    if (a.smooth) {
        for (int pass = 0; pass < 2; ++pass)
            timed(pass ? "k_chain_smoother_again" : "k_chain_smoother", s, [&] {
                if (tv) hipLaunchKernelGGL((k_chain_smoother_tv<T, NX>), grid, wave, 0, s, a, pass);
                else hipLaunchKernelGGL((k_chain_smoother_ti<T, NX>), pass ? grid : more, wave, 0, s, a, pass, pass ? 0 : writers);
            });
        timed("k_chain_check", s, [&] { hipLaunchKernelGGL((k_chain_check<true>), grid, wave, 0, s, a); });
    }
    return hipGetLastError();
}

template <typename T, int NX>
hipError_t run_ny(const Args& a, bool tv, hipStream_t s) {
    switch (a.ny) {
        case 1: return run<T, NX, 1>(a, tv, s);
        case 2: return run<T, NX, 2>(a, tv, s);
        case 3: return run<T, NX, 3>(a, tv, s);
        default: return run<T, NX, 4>(a, tv, s);
    }
}
template <typename T>
hipError_t run_nx(const Args& a, bool tv, hipStream_t s) {
    return a.nx == 3 ? run_ny<T, 3>(a, tv, s) : run_ny<T, 4>(a, tv, s);
}

}  // namespace

// Time-varying models.  Filter + smoother, general scan and chains, us:
//                                                   FP64            mixed (FP32 elements)
//   nx = 4, ny = 2, CV, q / r = 4, 2^18 steps       366, 274        261, 285
//                   2^19                            686, 337        534, 333
//                   2^20                            1277, 480       1043, 456
//   nx = 4, ny = 2, a mixture of models, 2^18       375, 302        268, 310
//                   2^19                            684, 389        535, 390
//   nx = 3, ny = 1, 2^18                            258, 262        185, 265
//                   2^19                            540, 310        394, 315
//   nx = 4, ny = 4, 2^18                            462, 417        354, 420
//                   2^19                            869, 536        669, 543
//   nx = 2, ny = 1, 2^20                            551, 934        465, 860 (an earlier form of the chains)
// (the chains' time hardly depends on nx, the general scan's does).  A model that the
// pilots give up costs 23 us more than the general scan alone, one that they let by
// and that does not forget in time 30 %.  Packed
// sequences: long enough on average that most chains are full ones.
// A model per sequence (nx = 4, ny = 2, CV models): the head and the tail of a
// sequence cost as much as about 1500 of its other steps, and a bundle with a
// model that settles too late goes back to the scan after 18 to 31 us:
//   64 sequences, 890 k steps (on the line)         324, 333        211 (the scan)
//                 the filter alone                  170, 133        114, 130 (below its line)
//   300,          2.46 M                            762, 469        445, 390
//                 the filter alone                  358, 180        244, 154
//   1024,         3.17 M                            968, 534        577, 414
//   1024,         8.29 M                            2039, 834       1224, 549
bool applies(int nx, int ny, int32_t B, int64_t total, bool mixed, bool tv, bool smooth) {
    if (nx < 3 || nx > 4 || ny > 4) return false;
    if (tv) return total >= (mixed ? 1 << 19 : 1 << 18) && total / B >= 512;
    return total - 1536 * (int64_t)B >= (int64_t)(mixed ? 2 : 1) * (smooth ? 3 << 18 : 1 << 19);
}

bool layout(Args& a, char* base, size_t bytes, bool tv) {
    // time-varying: a constant-velocity model sampled at 0.05 to 0.15 s forgets to
    // rounding in 190 to 210 steps where q / r = 4 s^-3, in 230 where 2.4, 370 where
    // 0.4, 600 where 0.04: those are met by the second pass, if at all, which starts
    // a.l + a.warm steps before.  Else the setup knows
    a.warm = 208;
    a.l = tv ? (a.total + 4095) / 4096 : std::max<int64_t>(64, (a.total + 12287) / 12288);
    // what has not been forgotten after a.warm steps falls on as it did until then
    a.near = std::exp2(-2.0 * 50.0 * (double)a.warm / (double)(a.warm + a.l));
    const int group = tv ? kAhead : kLong;            // chains start and end with a group of steps
    a.l = (a.l + group - 1) / group * group;
    a.max_chains = (a.total + a.l - 1) / a.l + (a.offsets ? a.B : 0);
    char* p = base;
    auto take = [&](int64_t words) {
        double* q = reinterpret_cast<double*>(p);
        p += ((size_t)words * sizeof(double) + 255) & ~size_t(255);
        return q;
    };
    a.first = reinterpret_cast<int64_t*>(take(a.B + 1));
    a.sequence = a.offsets ? reinterpret_cast<int*>(take((a.max_chains + 1) / 2)) : nullptr;
    a.model = tv ? nullptr : take((int64_t)a.B * kModel);
    a.forgets = reinterpret_cast<int*>(take((a.max_chains + 1) / 2));
    a.head = tv ? nullptr : reinterpret_cast<int*>(take(a.B));
    a.entry = take(a.max_chains * kState);
    a.end[0] = take(a.max_chains * kState);
    a.end[1] = take(a.max_chains * kState);
    return (size_t)(p - base) <= bytes;
}

hipError_t launch(const Args& a, bool mixed, bool tv, hipStream_t s) {
    return mixed ? run_nx<float>(a, tv, s) : run_nx<double>(a, tv, s);
}

}  // namespace chains
}  // namespace pks
