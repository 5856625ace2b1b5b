// chains.hip -- filter and smoother by overlapped chains (see chains.hpp).
//
// A wave runs four chains.  Every matrix of a chain, 4 x 4, is one double per
// lane (nx, ny <= 4, padded with zeros): lane j + 4 b + 16 i holds X(i, j) of
// chain b, the operand and result layout of v_mfma_f64_4x4x4_4b_f64, which
// multiplies four pairs of such tiles: mm(X, Y) = X^T Y.  Vectors are column 0.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "chains.hpp"
#include "tile16.hpp"

namespace pks {
namespace chains {

namespace {

constexpr int kAhead = 4;            // steps of a group; their loads are issued a group or two before
constexpr double kSame = 5.684341886080802e-14;       // 2^-44

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
    __device__ __forceinline__ double get(int s) const {
        if constexpr (sizeof(T) == 8) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)at, (int)(s * step), 0);
            return __builtin_bit_cast(double, v);
        } else {
            return (double)__builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)at, (int)(s * step), 0));
        }
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
        int lo = 0, hi = a.B;                // first[lo] <= c < first[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (a.first[mid] <= x.c) lo = mid; else hi = mid;
        }
        x.b = lo;
        x.lo = a.offsets[lo];
        x.hi = a.offsets[lo + 1];
        before = a.first[lo];
    }
    x.s = x.lo + (x.c - before) * a.l;
    x.e = min(x.s + a.l, x.hi);
    return x;
}

// moments (P, m) and (P2, m2) agree: differences against the standard deviations,
// the mean's against the size of the whole mean as well (its rounding is)
__device__ __forceinline__ bool agree(double P, double m, double P2, double m2, const Lane& t) {
    const double D = t.i == t.j ? P2 : 0.0, di = mm(D, 1.0), dj = mm(1.0, D);
    const double zz = t.j == 0 && di > 0.0 ? m2 / sqrt(di) : 0.0;
    const double z = col<0>(row<0>(mm(zz, zz), t));
    const double dP = P - P2, dm = t.j == 0 ? m - m2 : 0.0;
    const bool same = dP * dP <= kSame * kSame * di * dj && dm * dm <= kSame * kSame * di * (1.0 + z);
    const unsigned long long off = __ballot(!same);
    return (off & (0x000f000f000f000full << (4 * t.b))) == 0;
}

// ---------------------------------------------------------------------------
// the steps
// ---------------------------------------------------------------------------
struct Row {
    double FT, Q, HT, R, u, y;               // y less d
};
template <int NY>
__device__ __forceinline__ void filter_step(const Row& x, const Lane& t, double& m, double& P, bool& ok) {
    const double W = mm(P, x.FT), mp = mm(x.FT, m, x.u);
    const double Pp = mm(x.FT, W, x.Q);                       // F P F^T + Q
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
    ET = mm(inv<NX>(Pp, t, ok), FP);
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

// ---------------------------------------------------------------------------
// The flags, and the chains of every packed sequence.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_chain_setup(Args a) {
    const int lane = threadIdx.x;
    if (lane == 0) {
        if (a.reset || a.status[1] != kStatusMagic) {
            a.status[0] = kStatusOk;
            a.status[1] = kStatusMagic;
        }
        a.ctl[0] = 1;
    }
    if (!a.offsets) return;
    int64_t before = 0;
    for (int b0 = 0; b0 < a.B; b0 += 64) {
        const int b = b0 + lane;
        const int64_t own = b < a.B ? (a.offsets[b + 1] - a.offsets[b] + a.l - 1) / a.l : 0;
        int64_t inc = own;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t v = __shfl_up(inc, d, 64);
            if (lane >= d) inc += v;
        }
        if (b < a.B) a.first[b] = before + inc - own;
        before += __shfl(inc, 63, 64);
    }
    if (lane == 0) a.first[a.B] = before;
}

// ---------------------------------------------------------------------------
// The chains.  Bound by the rows of the model (F, Q, H, R: 368 bytes a step at
// nx = 4, ny = 2 with y), which the warm-up reads again, and by the latency of a
// step (six dependent products and the inverse of S: 0.33 us): 4096 chains, a
// wave per SIMD, balance the two.  nx = 4, ny = 2, FP64, 2^20 steps: the filter
// 208 us (4 TB/s), the smoother 205 us, where the block elements of the general
// scan took 464 us for the constants of every step and 760 us for the scans.
// ---------------------------------------------------------------------------
template <typename T, int NY>
__global__ __launch_bounds__(64) void k_chain_filter_tv(Args a, int pass) {
    if (pass && a.ctl[0] == 0) return;
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
        const bool same = agree(oP, om, P, m, t) || x.s == x.lo;
        if (same && x.live) {
            load_state(a.end[0], x.c, t, oP, om);
            store_state(a.end[1], x.c, t, oP, om);
        }
        todo = todo && !same;
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
    Row g[3][kAhead];
    auto fetch = [&](Row (&r)[kAhead]) {
#pragma unroll
        for (int q = 0; q < kAhead; ++q)
            r[q] = Row{rFT.get(q), rQ.get(q), rHT.get(q), rR.get(q), ru.get(q), ry.get(q) - rd.get(q)};
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
    auto use = [&](const Row (&r)[kAhead]) {
        if (k == s && todo) store_state(a.entry, x.c, t, P, m);
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const bool out = k + q < e && k + q >= s;
            bool fine = row_ok<NY>(r[q], t);
            filter_step<NY>(r[q], t, m, P, fine);
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
        const bool same = agree(oP, om, Ps, ms, t) || x.e == x.hi;
        if (same && x.live) {
            load_state(a.end[0], x.c, t, oP, om);
            store_state(a.end[1], x.c, t, oP, om);
        }
        todo = todo && !same;
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
        double FT, Q, u, m, P;
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
            smoother_gain<NX>(r[q].FT, r[q].Q, r[q].u, r[q].m, r[q].P, t, ET, Pp, mp, fine);
            const bool on = k + q < top, out = k + q < e && k >= s;
            double mn = ms, Pn = Ps;
            smoother_step(ET, Pp, mp, r[q].m, r[q].P, mn, Pn);
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
    const bool same = agree(P, m, P2, m2, t);
    if (x.live && !edge && !same) a.ctl[0] = 0;
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
hipError_t run(const Args& a, hipStream_t s) {
    const dim3 grid((unsigned)((a.max_chains + 3) / 4)), wave(64);
    timed("k_chain_setup", s, [&] { hipLaunchKernelGGL(k_chain_setup, dim3(1), wave, 0, s, a); });
    for (int pass = 0; pass < 2; ++pass)
        timed(pass ? "k_chain_filter_again" : "k_chain_filter", s,
              [&] { hipLaunchKernelGGL((k_chain_filter_tv<T, NY>), grid, wave, 0, s, a, pass); });
    timed("k_chain_check", s, [&] { hipLaunchKernelGGL((k_chain_check<false>), grid, wave, 0, s, a); });
    if (a.smooth) {
        for (int pass = 0; pass < 2; ++pass)
            timed(pass ? "k_chain_smoother_again" : "k_chain_smoother", s,
                  [&] { hipLaunchKernelGGL((k_chain_smoother_tv<T, NX>), grid, wave, 0, s, a, pass); });
        timed("k_chain_check", s, [&] { hipLaunchKernelGGL((k_chain_check<true>), grid, wave, 0, s, a); });
    }
    return hipGetLastError();
}

template <typename T, int NX>
hipError_t run_ny(const Args& a, hipStream_t s) {
    switch (a.ny) {
        case 1: return run<T, NX, 1>(a, s);
        case 2: return run<T, NX, 2>(a, s);
        case 3: return run<T, NX, 3>(a, s);
        default: return run<T, NX, 4>(a, s);
    }
}
template <typename T>
hipError_t run_nx(const Args& a, hipStream_t s) {
    return a.nx == 3 ? run_ny<T, 3>(a, s) : run_ny<T, 4>(a, s);
}

}  // namespace

// Filter + smoother, general scan and chains, us:       FP64        mixed (FP32 elements)
//   nx = 4, ny = 2, 2^18 steps                        371, 249      273, 259
//                   2^19                              677, 305      531, 312
//   nx = 3, ny = 1, 2^18                              256, 235      192, 241
//                   2^19                              543, 280      379, 286
//   nx = 4, ny = 4, 2^18                              459, 331      360, 369
//   nx = 2, ny = 1, 2^20                              551, 934      465, 860
// (the chains' time hardly depends on nx, the general scan's does).  Packed
// sequences: long enough on average that most chains are full ones.
bool applies(int nx, int ny, int32_t B, int64_t total, bool mixed) {
    return nx >= 3 && nx <= 4 && ny <= 4 && total >= (mixed ? 1 << 19 : 1 << 18) && total / B >= 512;
}

bool layout(Args& a, char* base, size_t bytes) {
    // CV models of all step sizes in use agree to rounding after 100 to 180 steps
    a.warm = 192;
    a.l = (a.total + 4095) / 4096;                    // (at least 64)
    a.l = (a.l + kAhead - 1) / kAhead * kAhead;       // chains start and end with a group of steps
    a.max_chains = (a.total + a.l - 1) / a.l + (a.offsets ? a.B : 0);
    char* p = base;
    auto take = [&](int64_t words) {
        double* q = reinterpret_cast<double*>(p);
        p += ((size_t)words * sizeof(double) + 255) & ~size_t(255);
        return q;
    };
    a.first = reinterpret_cast<int64_t*>(take(a.B + 1));
    a.entry = take(a.max_chains * kState);
    a.end[0] = take(a.max_chains * kState);
    a.end[1] = take(a.max_chains * kState);
    return (size_t)(p - base) <= bytes;
}

hipError_t launch(const Args& a, bool mixed, hipStream_t s) {
    return mixed ? run_nx<float>(a, s) : run_nx<double>(a, s);
}

}  // namespace chains
}  // namespace pks
