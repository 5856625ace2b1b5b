// steady.hip -- filter and smoother of a time-invariant model with settled
// covariances (see steady.hpp), nx, ny <= 16: setup kernels on register tiles,
// and the recursions of the means with 16 chains of steps in the columns of a
// tile.
//
// Launches: k_st_double (one wave: doubling, settled gains, powers),
// k_st_tables (a wave per run of kRun head or tail steps), then the means:
// reduce (chains from zero), top (a sequence's tiles), down, each for the
// filter and, backwards, for the smoother.  The filter reduce and the smoother
// down-sweep also write the covariances, which do not wait for the means.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "steady_ops.hpp"

namespace pks {
namespace steady {

namespace {

// (M^T)^-1 for M = I + C J given the tiles of C and J: unpivoted, refined where the
// residual is not rounding, with partial pivoting where it is not small
template <int KX>
__device__ __forceinline__ f64x4 inv_ijc(const f64x4& C, const f64x4& J, const f64x4& I, double* st, int n, bool& ok) {
    const f64x4 MT = mm<KX>(J, C, I);
    bool good = true;
    f64x4 NT = inv_np<4 * KX, false>(MT, good);
    const f64x4 R = mm<KX>(mm<KX>(C, J, I), NT);
    double dev = 0.0;
#pragma unroll
    for (int v = 0; v < KX; ++v) dev = fmax(dev, fabs(R[v] - I[v]));
    if (!good || __any(!(dev <= kExact))) {
        if (!good || __any(!(dev <= kSmall))) return inv_piv(MT, n, st, ok);
        NT = mm<KX>(tr(NT, st), I - R, NT);
    }
    return NT;
}

struct Model16 {
    f64x4 F, FT, Q, HT, R, u, d;
    int n, m;
};
__device__ __forceinline__ Model16 load_model(const Args& a) {
    Model16 x;
    const int n = x.n = a.nx, m = x.m = a.ny;
    x.F = load_tile(a.F, n, n, n);
    x.FT = load_tile_t(a.F, n, n, n);
    x.Q = pad_eye(load_tile(a.Q, n, n, n), n);
    x.HT = load_tile_t(a.H, m, n, n);
    x.R = pad_eye(load_tile(a.R, m, m, m), m);
    x.u = a.u ? load_vec(a.u, n) : zero4();
    x.d = a.d ? load_vec(a.d, m) : zero4();
    return x;
}

// S^-1 X given the inverse Si of the symmetric S, refined where the residual is not
// rounding, after which the quotient is as good as a factorisation's (a product with
// an inverse alone loses the digits of S's condition: smoothed covariances of the
// first steps behind a prior of 1e4 I were 8e-9 off, 2e-11 by the Cholesky solves of
// the scan)
template <int KS>
__device__ __forceinline__ f64x4 solve(const f64x4& S, const f64x4& Si, const f64x4& X) {
    const f64x4 q = mm<KS>(Si, X), r = X - mm<KS>(S, q);
    bool off = false;
#pragma unroll
    for (int v = 0; v < 4; ++v) off |= !(fabs(r[v]) <= kExact * fabs(X[v]));
    return __any(off) ? mm<KS>(Si, r, q) : q;
}
// FP = F P and the predicted covariance F P F^T + Q (the identity beyond nx)
template <int KX>
__device__ __forceinline__ void predict(const Model16& x, const f64x4& P, double* st, f64x4& FP, f64x4& Pm) {
    FP = mm<KX>(x.FT, P);
    Pm = symt(mm<KX>(x.FT, tr(FP, st), x.Q), zero4(), st);
}
// the update: K^T, Phi and c, and the new P (zero beyond nx)
template <int KX, int KY>
__device__ __forceinline__ void update(const Model16& x, const f64x4& Pm, double* st, bool& ok, f64x4& P, f64x4& Kt,
                                       f64x4& Phi, f64x4& c) {
    const f64x4 HP = mm<KX>(x.HT, Pm);
    const f64x4 S = symt(mm<KX>(x.HT, tr(HP, st), x.R), zero4(), st);
    Kt = solve<KY>(S, inv_np<4 * KY, true>(S, ok), HP);          // S^-1 H Pm
    const f64x4 nKt = -Kt;
    P = symt(mm<KY>(nKt, HP, Pm), zero4(), st);
    const int li = lane_i(), lk = lane_k();
#pragma unroll
    for (int v = 0; v < 4; ++v)
        if (4 * v + lk == li && li >= x.n) P[v] = 0.0;
    Phi = mm<KY>(nKt, mm<KX>(x.HT, x.F), x.F);
    c = mm<KY>(nKt, mm<KX>(x.HT, x.u, x.d), x.u);
}
// smoothing element (Lemma 3, matrix parts) of a step with filtered covariance
// P: the tiles of E^T and L
template <int KX>
__device__ __forceinline__ void smooth_elem(const f64x4& P, const f64x4& FP, const f64x4& Pm, double* st, bool& ok,
                                            f64x4& ET, f64x4& L) {
    ET = solve<KX>(Pm, inv_np<4 * KX, true>(Pm, ok), FP);
    const f64x4 EFP = mm<KX>(ET, FP), EFPt = tr(EFP, st);
#pragma unroll
    for (int v = 0; v < 4; ++v) L[v] = P[v] - 0.5 * (EFP[v] + EFPt[v]);
}
// E L E^T + add, E by the tile of E^T
template <int KX>
__device__ __forceinline__ f64x4 ele(const f64x4& ET, const f64x4& L, const f64x4& add, double* st) {
    return symt(mm<KX>(mm<KX>(L, ET), ET), add, st);
}
// whether what a covariance P adds to C by way of A, A P A^T, is at most f of C in
// every variance (AT: the tile of A^T)
template <int KX>
__device__ __forceinline__ bool negligible(const f64x4& AT, const f64x4& P, const f64x4& C, double f, int n) {
    return diagonal_below(mm<KX>(AT, mm<KX>(P, AT)), C, f, n);
}
template <int KX>
__device__ __forceinline__ bool meets(const f64x4& x, const f64x4& y) {
    const f64x4 d = diagonal(y);
    return steady::meets(x, y, mm<KX>(d, ones()), mm<KX>(ones(), d));
}
__device__ __forceinline__ void store_gain(double* X, const f64x4& K, int n, int m) {
    const int li = lane_i(), lk = lane_k();
#pragma unroll
    for (int v = 0; v < 4; ++v)
        if (4 * v + lk < n && li < m) X[(4 * v + lk) * m + li] = K[v];
}

// ---------------------------------------------------------------------------
// Doubling.  One wave, because every combine needs the one before: it is bound
// by the latency of about log2 n dependent combines (an inverse each).
// ---------------------------------------------------------------------------
template <int KX, int KY>
__global__ __launch_bounds__(64) void k_st_double(Args a) {
    __shared__ double st[kStage];
    const int n = a.nx, n2 = n * n, lane = threadIdx.x;
    if (lane == 0) {
        if (a.reset || a.status[1] != kStatusMagic) {
            a.status[0] = kStatusOk;
            a.status[1] = kStatusMagic;
        }
        a.ctl[0] = 0;
    }
    const Model16 x = load_model(a);
    const f64x4 I = eye(), P0 = load_tile(a.P0, n, n, n);
    bool ok = true;
    // the element of one step (Lemma 1)
    f64x4 A, C, J;
    {
        const f64x4 Q = load_tile(a.Q, n, n, n);
        const f64x4 T1 = mm<KX>(x.HT, Q);
        const f64x4 S = symt(mm<KX>(tr(T1, st), x.HT, x.R), zero4(), st);
        const f64x4 Si = inv_np<4 * KY, true>(S, ok);
        const f64x4 nKt = -mm<KY>(Si, T1), G = mm<KX>(x.HT, x.F);
        J = symt(mm<KY>(G, mm<KY>(Si, G)), zero4(), st);
        A = mm<KY>(nKt, G, x.F);
        C = symt(mm<KY>(nKt, T1, Q), zero4(), st);
    }
    store_tile(a.powF, A, n);
    store_tile(a.powF + n2, C, n);
    store_tile(a.powF + 2 * n2, J, n);
    int lf = 0, le = 0;
    bool settled = false;
    f64x4 AT = tr(A, st);
#pragma unroll 1
    for (int l = 1; (1 << l) <= a.N && ok; ++l) {
        const f64x4 NT = inv_ijc<KX>(C, J, I, st, n, ok);
        const f64x4 X1 = mm<KX>(NT, A), X3 = mm<KX>(NT, C), JA = mm<KX>(J, A);
        A = mm<KX>(AT, X1);
        C = symt(mm<KX>(AT, mm<KX>(X3, AT)), C, st);
        AT = tr(A, st);
        J = symt(mm<KX>(X1, JA), J, st);
        double* rec = a.powF + (int64_t)l * 3 * n2;
        store_tile(rec, A, n);
        store_tile(rec + n2, C, n);
        store_tile(rec + 2 * n2, J, n);
        lf = l;
        if ((1 << l) >= kRun && negligible<KX>(AT, P0 + C, C, kTiny, n)) {
            settled = true;
            break;
        }
    }
    if (!(settled && ok)) return;
    // the settled gains
    const f64x4 P = C;
    f64x4 FP, Pm, Kt, Phi, c, ET, L, Pn;
    predict<KX>(x, P, st, FP, Pm);
    smooth_elem<KX>(P, FP, Pm, st, ok, ET, L);
    update<KX, KY>(x, Pm, st, ok, Pn, Kt, Phi, c);
    store_tile(a.star + star_P(n, x.m), P, n);
    store_tile(a.star + star_Phi(n, x.m), Phi, n);
    store_gain(a.star + star_K(n, x.m), tr(Kt, st), n, x.m);
    store_vec(a.star + star_c(n, x.m), c, n);
    store_tile(a.star + star_E(n, x.m), tr(ET, st), n);
    store_tile(a.star + star_L(n, x.m), L, n);
    // smoothing elements of 2^l settled steps
    settled = false;
#pragma unroll 1
    for (int l = 0; (1 << l) <= a.N && ok; ++l) {
        f64x4 E = tr(ET, st);
        if (l > 0) {
            L = ele<KX>(ET, L, L, st);
            ET = mm<KX>(E, ET);                                  // (E E)^T
            E = tr(ET, st);
        }
        store_tile(a.powE + (int64_t)l * 2 * n2, E, n);
        store_tile(a.powE + (int64_t)l * 2 * n2 + n2, L, n);
        le = l;
        if ((1 << l) >= kRun && negligible<KX>(ET, P, L, kTiny, n)) {
            settled = true;
            break;
        }
    }
    if (!(settled && ok)) return;
    store_tile(a.star + star_Ps(n, x.m), L, n);
    // the chain blocks of every sequence beyond the head
    const int nh = 1 << (lf > le ? lf : le);
    const int64_t per = (int64_t)kBlockChains << a.pL;
    int64_t before = 0;
    for (int b0 = 0; b0 < a.B; b0 += 64) {
        const int b = b0 + lane;
        int64_t t = 0;
        if (b < a.B) {
            const int64_t len = a.offsets ? a.offsets[b + 1] - a.offsets[b] : a.total;
            if (len > nh) t = (len - nh + per - 1) / per;
        }
        int64_t inc = t;
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) {
            const int64_t o = __shfl_up(inc, s, 64);
            if (lane >= s) inc += o;
        }
        if (b < a.B) a.blk_off[b] = before + inc - t;
        before += __shfl(inc, 63, 64);
    }
    if (lane == 0) {
        a.blk_off[a.B] = before;
        a.ctl[1] = lf;
        a.ctl[2] = le;
        a.ctl[0] = nh;
    }
}

// ---------------------------------------------------------------------------
// Head and tail tables: wave i forms kRun consecutive head steps (covariance,
// gains, smoothing elements) from the covariance after i kRun steps, which the
// doubled elements give in one carry per set bit; waves beyond the head's form
// kRun tail steps the same way, and the last two the powers Phi^(L 2^i) and
// E^(L 2^i).  Bound by the latency of those dependent inverses: a short run per
// wave, as many waves as there are runs.
// ---------------------------------------------------------------------------
template <int KX, int KY>
__global__ __launch_bounds__(64) void k_st_tables(Args a) {
    __shared__ double st[kStage];
    const int nh = a.ctl[0];
    if (nh == 0) return;
    const int nrun = nh / kRun;
    const int n = a.nx, n2 = n * n, m = a.ny;
    int blk = blockIdx.x;
    if (blk < 2) {                           // powers
        if (blk == 1 && !a.smooth) return;
        const double* src = a.star + (blk == 0 ? star_Phi(n, m) : star_E(n, m));
        double* out = blk == 0 ? a.mpF : a.mpE;
        f64x4 M = load_tile(src, n, n, n), MT = load_tile_t(src, n, n, n);
#pragma unroll 1
        for (int p = 0; p < a.pL + kPowers; ++p) {
            if (p >= a.pL) store_tile(out + (int64_t)(p - a.pL) * n2, M, n);
            M = mm<KX>(MT, M);
            MT = tr(M, st);
        }
        return;
    }
    blk -= 2;
    if (blk >= (a.smooth ? 2 : 1) * nrun) return;
    const f64x4 I = eye();
    bool ok = true;
    if (blk >= nrun) {                       // tail: Ps j steps before the last
        const int j0 = (blk - nrun) * kRun;
        f64x4 Ps;
        if (j0 >> a.ctl[2]) {
            Ps = load_tile(a.star + star_Ps(n, m), n, n, n);
        } else {
            Ps = load_tile(a.star + star_P(n, m), n, n, n);
#pragma unroll 1
            for (int l = 0; (j0 >> l) != 0; ++l)
                if ((j0 >> l) & 1) {
                    const double* rec = a.powE + (int64_t)l * 2 * n2;
                    Ps = ele<KX>(load_tile_t(rec, n, n, n), Ps, load_tile(rec + n2, n, n, n), st);
                }
        }
        const f64x4 ET = load_tile_t(a.star + star_E(n, m), n, n, n), L = load_tile(a.star + star_L(n, m), n, n, n);
#pragma unroll 1
        for (int j = j0; j < j0 + kRun; ++j) {
            store_tile(a.tTail + (int64_t)j * n2, Ps, n);
            Ps = ele<KX>(ET, Ps, L, st);
        }
        if (j0 + kRun == 1 << a.ctl[2] && !meets<KX>(Ps, load_tile(a.star + star_Ps(n, m), n, n, n)) && threadIdx.x == 0)
            atomicExch(&a.ctl[0], 0);
        return;
    }
    const int k0 = blk * kRun;
    const Model16 x = load_model(a);
    f64x4 P = load_tile(a.P0, n, n, n);
    const f64x4 Pstar = load_tile(a.star + star_P(n, m), n, n, n);
    const f64x4 AnT = load_tile_t(a.powF + (int64_t)a.ctl[1] * 3 * n2, n, n, n);       // of the steps that it takes to settle
    if (k0 >> a.ctl[1]) {
        P = Pstar;
    } else {
#pragma unroll 1
        for (int l = 0; (k0 >> l) != 0; ++l)
            if ((k0 >> l) & 1) {
                const double* rec = a.powF + (int64_t)l * 3 * n2;
                const f64x4 J = load_tile(rec + 2 * n2, n, n, n), AT = load_tile_t(rec, n, n, n);
                const f64x4 C = load_tile(rec + n2, n, n, n);
                const f64x4 X3 = mm<KX>(inv_ijc<KX>(P, J, I, st, n, ok), P);
                P = symt(mm<KX>(AT, mm<KX>(X3, AT)), C, st);
            }
    }
    f64x4 EaT = I, La = zero4(), Pa = I;     // smoothing element and Phi of the run's steps
#pragma unroll 1
    for (int k = k0; k < k0 + kRun; ++k) {
        f64x4 FP, Pm, Kt, Phi, c;
        predict<KX>(x, P, st, FP, Pm);
        if (a.smooth) {                      // of step k - 1, whose covariance P is
            f64x4 ET, L;
            smooth_elem<KX>(P, FP, Pm, st, ok, ET, L);
            if (k > 0) {
                const f64x4 E = tr(ET, st);
                store_tile(a.tE + (int64_t)(k - 1) * n2, E, n);
                store_tile(a.tL + (int64_t)(k - 1) * n2, L, n);
                La = ele<KX>(EaT, L, La, st);
                EaT = mm<KX>(E, EaT);        // (E_a E)^T
            }
        }
        update<KX, KY>(x, Pm, st, ok, P, Kt, Phi, c);
        ok = ok && negligible<KX>(AnT, P, Pstar, kSpare * kTiny, n);
        Pa = mm<KX>(tr(Phi, st), Pa);
        store_tile(a.tP + (int64_t)k * n2, P, n);
        store_tile(a.tPhi + (int64_t)k * n2, Phi, n);
        store_gain(a.tK + (int64_t)k * n * m, tr(Kt, st), n, m);
        store_vec(a.tc + (int64_t)k * n, c, n);
    }
    store_tile(a.runPhi + (int64_t)blk * n2, Pa, n);
    if (a.smooth) {
        store_tile(a.runE + (int64_t)blk * n2, tr(EaT, st), n);
        store_tile(a.runL + (int64_t)blk * n2, La, n);
        if (k0 + kRun == nh) {               // E of the head's last step, whose covariance has settled
            store_tile(a.tE + (int64_t)(nh - 1) * n2, load_tile(a.star + star_E(n, m), n, n, n), n);
            store_tile(a.tL + (int64_t)(nh - 1) * n2, load_tile(a.star + star_L(n, m), n, n, n), n);
        }
    }
    if (k0 + kRun == 1 << a.ctl[1]) ok = ok && meets<KX>(P, Pstar);
    if (!ok && threadIdx.x == 0) atomicExch(&a.ctl[0], 0);
}

// Smoothed covariances of the head, backwards from the settled one: the value
// at the last step of every run.  The waves of a workgroup compose a chunk of
// runs each, one wave takes the chunks one after another, and the waves then
// replay their runs from the values that enter their chunks.
constexpr int kTopWaves = 16;
template <int KX>
__device__ __forceinline__ void head_runs(const Args& a, int nh, double* st, double* ce, double* cl) {
    const int n = a.nx, n2 = n * n, nrun = nh / kRun, wave = threadIdx.x >> 6;
    const int q = (nrun + kTopWaves - 1) / kTopWaves;
    // chunk w holds the runs nrun - 1 - w q, ... downwards
    const int hi = nrun - 1 - wave * q, lo = hi - q + 1 > 0 ? hi - q + 1 : 0;
    if (hi >= 0) {
        f64x4 ET = load_tile_t(a.runE + (int64_t)hi * n2, n, n, n), L = load_tile(a.runL + (int64_t)hi * n2, n, n, n);
#pragma unroll 1
        for (int i = hi - 1; i >= lo; --i) {                      // (run i) (x) (what is later)
            const f64x4 EiT = load_tile_t(a.runE + (int64_t)i * n2, n, n, n);
            L = ele<KX>(EiT, L, load_tile(a.runL + (int64_t)i * n2, n, n, n), st);
            ET = mm<KX>(tr(ET, st), EiT);                         // (E_i E)^T
        }
        put_tile(ce + wave * kTile, ET);
        put_tile(cl + wave * kTile, L);
    }
    __syncthreads();
    if (wave == 0) {
        f64x4 Ps = load_tile(a.star + star_Ps(n, a.ny), n, n, n);
#pragma unroll 1
        for (int w = 0; w * q < nrun; ++w) {
            const f64x4 ET = get_tile(ce + w * kTile), L = get_tile(cl + w * kTile);
            put_tile(cl + w * kTile, Ps);
            Ps = ele<KX>(ET, Ps, L, st);
        }
    }
    __syncthreads();
    if (hi >= 0) {
        f64x4 Ps = get_tile(cl + wave * kTile);
#pragma unroll 1
        for (int i = hi; i >= lo; --i) {
            store_tile(a.runC + (int64_t)i * n2, Ps, n);
            Ps = ele<KX>(load_tile_t(a.runE + (int64_t)i * n2, n, n, n), Ps, load_tile(a.runL + (int64_t)i * n2, n, n, n), st);
        }
    }
}
// and at the other steps of run i
template <int KX>
__device__ __forceinline__ void head_fill(const Args& a, int i, double* st) {
    const int n = a.nx, n2 = n * n;
    f64x4 Ps = load_tile(a.runC + (int64_t)i * n2, n, n, n);
    int k = i * kRun + kRun - 1;
    store_tile(a.tHead + (int64_t)k * n2, Ps, n);
    for (; k > i * kRun; --k) {
        Ps = ele<KX>(load_tile_t(a.tE + (int64_t)(k - 1) * n2, n, n, n), Ps, load_tile(a.tL + (int64_t)(k - 1) * n2, n, n, n), st);
        store_tile(a.tHead + (int64_t)(k - 1) * n2, Ps, n);
    }
}

// A sequence shorter than 2 n: its smoothed head covariances depend on its
// length and are folded one by one (Lemma 4) from its own last ones.
template <typename R, int KX>
__device__ __forceinline__ void short_head(const Args& a, int nh, int b, double* st) {
    const int n = a.nx, n2 = n * n;
    const SeqR q = seq_of(a, b);
    const int64_t len = q.end - q.start;
    if (len >= 2 * nh || len < 1) return;
    R* out = static_cast<R*>(a.Ps) + q.start * n2;
    int64_t k;
    f64x4 Ps;
    if (len >= nh) {
        k = nh - 1;
        Ps = load_tile(a.tTail + (len - nh) * n2, n, n, n);
    } else {
        k = len - 1;
        Ps = load_tile(a.tP + k * n2, n, n, n);
        store_tile(out + k * n2, Ps, n);
    }
    f64x4 ETn = load_tile_t(a.tE + (k > 0 ? k - 1 : 0) * n2, n, n, n), Ln = load_tile(a.tL + (k > 0 ? k - 1 : 0) * n2, n, n, n);
    for (; k > 0; --k) {
        const f64x4 ET = ETn, L = Ln;
        const int64_t kn = k > 1 ? k - 2 : 0;
        ETn = load_tile_t(a.tE + kn * n2, n, n, n);
        Ln = load_tile(a.tL + kn * n2, n, n, n);
        Ps = ele<KX>(ET, Ps, L, st);
        store_tile(out + (k - 1) * n2, Ps, n);
    }
}

// ---------------------------------------------------------------------------
// Means: 16 chains (or 16 sequences' heads) in the columns of a tile, L steps
// each, so that a step of 16 chains is KX + KY MFMAs.  Above the tiles the
// chains' affine maps are scanned with the powers of one matrix: 16 chains of
// a tile, the 4 tiles of a workgroup, 16 workgroups, and those one after
// another.
// ---------------------------------------------------------------------------
// inclusive scan over the columns with the matrix M whose powers 1, 2, 4, 8
// are at mp: X_c <- X_c + M X_{c-1} + M^2 X_{c-2} + ... (UP; else over c + 1, ...)
template <int KX, bool UP>
__device__ __forceinline__ f64x4 column_scan(f64x4 X, const double* mp, int n) {
    const int n2 = n * n;
    const f64x4 p0 = load_op<KX>(mp, n, n), p1 = load_op<KX>(mp + n2, n, n);
    const f64x4 p2 = load_op<KX>(mp + 2 * n2, n, n), p3 = load_op<KX>(mp + 3 * n2, n, n);
    X = mm<KX>(p0, shift<UP, 1, KX>(X), X);
    X = mm<KX>(p1, shift<UP, 2, KX>(X), X);
    X = mm<KX>(p2, shift<UP, 4, KX>(X), X);
    return mm<KX>(p3, shift<UP, 8, KX>(X), X);
}
// the value v (every column holds it) that enters at the first column (last,
// if not UP): column c gets M^c v
template <int KX, bool UP>
__device__ __forceinline__ f64x4 column_spread(const f64x4& v, const double* mp, int n) {
    f64x4 X;
    const bool edge = lane_i() == (UP ? 0 : 15);
#pragma unroll
    for (int i = 0; i < 4; ++i) X[i] = edge ? v[i] : 0.0;
    return column_scan<KX, UP>(X, mp, n);
}

// the chain of this lane's column
struct Chain {
    int64_t start, len;    // of its sequence
    int64_t k0;            // its first step, within the sequence
};
__device__ __forceinline__ Chain chain_of(const Args& a, int nh, int64_t blk, int wave) {
    Chain c;
    const int b = a.B > 1 ? seq_holding(a.blk_off, a.B, blk) : 0;
    const SeqR q = seq_of(a, b);
    c.start = q.start;
    c.len = q.end - q.start;
    c.k0 = nh + (((blk - a.blk_off[b]) * kBlockChains + wave * 16 + lane_i()) << a.pL);
    return c;
}

// m at the kRun steps of a head run, from X; rows[] gets the means as stored
template <typename R, int KX, int KY, bool STORE>
__device__ __forceinline__ f64x4 run_filter(const Args& a, const Head& h, int run, f64x4 X, f64x4 (&rows)[kRun]) {
    const int n = a.nx, m = a.ny;
    const R* y = static_cast<const R*>(a.y) + h.start * m;
    R* mo = static_cast<R*>(a.m) + h.start * n;
    f64x4 phi[kRun], gain[kRun];
#pragma unroll
    for (int j = 0; j < kRun; ++j) {
        const int k = run * kRun + j;
        phi[j] = load_op<KX>(a.tPhi + (int64_t)k * n * n, n, n);
        const f64x4 kk = load_op<KY>(a.tK + (int64_t)k * n * m, n, m);
        const f64x4 yk = k < h.len ? load_col<KY>(y + (int64_t)k * m, m) : zero4();
        gain[j] = mm<KY>(kk, yk, load_col<KX>(a.tc + (int64_t)k * n, n));
    }
#pragma unroll
    for (int j = 0; j < kRun; ++j) {
        const int k = run * kRun + j;
        X = mm<KX>(phi[j], X, gain[j]);
        if constexpr (STORE) {
#pragma unroll
            for (int v = 0; v < 4; ++v) rows[j][v] = double(R(X[v]));
            if (k < h.len) store_col<KX>(mo + (int64_t)k * n, X, n);
        }
    }
    return X;
}
// Smoothed means backwards over the steps of smoothing run i (k0 + 2 .. k0 - 1,
// k0 = i kRun), from Z at step k0 + 3; mk[j]: the filtered means of step k0 - 1 + j
template <typename R, int KX, bool STORE>
__device__ __forceinline__ f64x4 run_smoother(const Args& a, const Head& h, int run, f64x4 Z, const f64x4 (&mk)[kRun]) {
    const int n = a.nx, n2 = n * n;
    R* mo = static_cast<R*>(a.ms) + h.start * n;
    const f64x4 FT = load_op<KX>(a.F, n, n), u = a.u ? load_col<KX>(a.u, n) : zero4();
    f64x4 et[kRun], p[kRun];
#pragma unroll
    for (int j = 0; j < kRun; ++j) {
        const int k = run * kRun - 1 + j;
        et[j] = load_op<KX>(a.tE + (int64_t)(k > 0 ? k : 0) * n2, n, n);
        p[j] = mm<KX>(FT, mk[j], u);
    }
#pragma unroll
    for (int j = kRun - 1; j >= 0; --j) {
        const int k = run * kRun - 1 + j;
        if (k < 0) break;
        const f64x4 Zn = mm<KX>(et[j], Z - p[j], mk[j]);
#pragma unroll
        for (int v = 0; v < 4; ++v) Z[v] = k >= h.full ? 0.0 : (k == h.full - 1 ? mk[j][v] : Zn[v]);
        if constexpr (STORE)
            if (k < h.len) store_col<KX>(mo + (int64_t)k * n, Z, n);
    }
    return Z;
}

struct Grid {
    int64_t heads, extra, blocks;     // workgroups for head runs, for other table work, for chain blocks
};
constexpr int kWG = 256;              // four waves, a tile each

// waves of a launch that take head runs: (group of 16 sequences, run)
__device__ __forceinline__ bool head_wave(const Args& a, int nh, int64_t blk, int wave, int& group, int& run) {
    const int nrun = nh / kRun;
    const int64_t id = blk * 4 + wave;
    group = (int)(id / nrun);
    run = (int)(id % nrun);
    return group * 16 < a.B;
}

// chains of the filter from zero; head runs from zero; P
template <typename R, int KX, int KY>
__global__ __launch_bounds__(kWG) void k_st_filter_reduce(Args a, Grid g) {
    __shared__ __align__(16) R row[256];
    __shared__ double ag[4][16];
    const int nh = a.ctl[0];
    if (nh == 0) return;
    const int n = a.nx, m = a.ny, wave = threadIdx.x >> 6;
    int64_t blk = blockIdx.x;
    if (blk < g.heads) {
        int group, run;
        if (!head_wave(a, nh, blk, wave, group, run)) return;
        const Head h = head_of(a, nh, group);
        f64x4 rows[kRun];
        const f64x4 X = run_filter<R, KX, KY, false>(a, h, run, zero4(), rows);
        if (h.full > 0) store_col<KX>(run_vec(a, a.runB, h.b, run), X, n);
        return;
    }
    blk -= g.heads;
    if (blk >= g.blocks) {
        write_rows<R, false>(a, nh, blk - g.blocks, gridDim.x - g.heads - g.blocks, row);
        return;
    }
    if (blk >= a.blk_off[a.B]) return;
    const Chain c = chain_of(a, nh, blk, wave);
    const R* y = static_cast<const R*>(a.y) + c.start * m;
    const f64x4 PhiT = load_op<KX>(a.star + star_Phi(n, m), n, n), KT = load_op<KY>(a.star + star_K(n, m), n, m);
    const f64x4 cc = load_col<KX>(a.star + star_c(n, m), n);
    const int64_t last = c.len - 1;
    const int L = 1 << a.pL;
    f64x4 X = zero4();
    auto at = [&](int64_t k) { return load_col<KY>(y + (k < last ? k : last) * m, m); };
    f64x4 yy[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) yy[j] = at(c.k0 + j);
    for (int i = 0; i < L; i += 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const f64x4 yk = yy[j];
            yy[j] = at(c.k0 + i + j + 4);
            X = mm<KX>(PhiT, X, mm<KY>(KT, yk, cc));
        }
    }
    X = column_scan<KX, true>(X, a.mpF, n);
    if (lane_i() == 15) store_col<KX>(ag[wave], X, n);
    __syncthreads();
    const f64x4 M16 = load_op<KX>(a.mpF + (int64_t)4 * n * n, n, n);
    f64x4 V = zero4();
    for (int s = 0; s < wave; ++s) V = mm<KX>(M16, V, load_col<KX>(ag[s], n));
    const f64x4 pre = shift<true, 1, KX>(X) + column_spread<KX, true>(V, a.mpF, n);
    store_col<KX>(a.pre + ((blk * 4 + wave) * 16 + lane_i()) * n, pre, n);
    if (wave == 3) {
        V = mm<KX>(M16, V, load_col<KX>(ag[3], n));
        if (lane_i() == 0) store_col<KX>(a.agg + blk * n, V, n);
    }
}

// The blocks of one sequence: the mean that enters each of them, and the mean
// that enters each run of its head.  Waves scan groups of 16 blocks and compose
// chunks of head runs; one wave takes those one after another, and the waves
// spread what enters their groups and chunks.  REV: backwards (the smoother).
// One more workgroup forms the smoothed covariances of the head.
constexpr int kTopGroups = 64;        // a sequence has at most 32768 chains and a part of one: 33 groups of 1024
template <typename R, int KX, bool REV>
__global__ __launch_bounds__(64 * kTopWaves) void k_st_top(Args a) {
    __shared__ double ga[kTopGroups * 16], gc[kTopGroups * 16];
    __shared__ double cb[kTopWaves * 16], cm[kTopWaves * kTile];
    __shared__ double aux[REV ? 1 : kTopWaves * (kTile + kStage)];
    const int nh = a.ctl[0];
    if (nh == 0) return;
    const int n = a.nx, n2 = n * n, b = blockIdx.x, wave = threadIdx.x >> 6, li = lane_i();
    if constexpr (!REV) {
        if (b == a.B) {
            head_runs<KX>(a, nh, aux + kTopWaves * kTile + wave * kStage, aux, cm);
            return;
        }
    }
    const SeqR sq = seq_of(a, b);
    const int64_t len = sq.end - sq.start;
    const int64_t t0 = a.blk_off[b], nt = a.blk_off[b + 1] - t0;
    const int ng = (int)((nt + 15) / 16), nrun = nh / kRun, q = (nrun + kTopWaves - 1) / kTopWaves;
    const double* mp = (REV ? a.mpE : a.mpF) + (int64_t)6 * n2;
    auto blk_at = [&](int64_t i) { return REV ? t0 + nt - 1 - i : t0 + i; };
    auto run_at = [&](int i) { return REV ? nrun - 1 - i : i; };
    const double* runM = REV ? a.runE : a.runPhi;
    // groups of blocks
    for (int g = wave; g < ng; g += kTopWaves) {
        const int64_t i = (int64_t)g * 16 + li;
        f64x4 X = i < nt ? load_col<KX>(a.agg + blk_at(i) * n, n) : zero4();
        X = column_scan<KX, true>(X, mp, n);
        if (i < nt) store_col<KX>(a.car + blk_at(i) * n, shift<true, 1, KX>(X), n);
        if (li == 15) store_col<KX>(ga + g * 16, X, n);
    }
    // chunks of head runs: the affine map of runs i0 .. i1 - 1
    const int i0 = wave * q, i1 = i0 + q < nrun ? i0 + q : nrun;
    if (i0 < i1) {
        f64x4 M = load_tile(runM + (int64_t)run_at(i0) * n2, n, n, n);
        f64x4 V = load_col<KX>(run_vec(a, a.runB, b, run_at(i0)), n);
#pragma unroll 1
        for (int i = i0 + 1; i < i1; ++i) {
            const f64x4 op = load_op<KX>(runM + (int64_t)run_at(i) * n2, n, n);
            V = mm<KX>(op, V, load_col<KX>(run_vec(a, a.runB, b, run_at(i)), n));
            M = mm<KX>(op, M);
        }
        const int lk = lane_k();
#pragma unroll
        for (int v = 0; v < 4; ++v) cm[wave * kTile + (4 * v + lk) * 16 + li] = M[v];
        if (li == 0) store_col<KX>(cb + wave * 16, V, n);
    }
    __syncthreads();
    if (wave == 0) {
        const f64x4 MG = load_op<KX>(mp + (int64_t)4 * n2, n, n);
        auto chunks = [&](f64x4 X) {
            for (int w = 0; w * q < nrun; ++w) {
                const f64x4 V = load_col<KX>(cb + w * 16, n);
                if (li == 0) store_col<KX>(cb + w * 16, X, n);
                X = mm<KX>(load_op<KX>(cm + w * kTile, 16, 16), X, V);
            }
            return X;
        };
        auto groups = [&](f64x4 X) {
            for (int g = 0; g < ng; ++g) {
                const f64x4 V = load_col<KX>(ga + g * 16, n);
                if (li == 0) store_col<KX>(gc + g * 16, X, n);
                X = mm<KX>(MG, X, V);
            }
            return X;
        };
        if constexpr (!REV) {
            groups(chunks(load_col<KX>(a.m0, n)));
        } else {
            // the last group is filled up with blocks that add nothing and still
            // multiply: the mean at the first step beyond the head comes from
            // what enters the sequence's first block instead
            groups(zero4());
        }
    }
    __syncthreads();
    for (int g = wave; g < ng; g += kTopWaves) {
        const int64_t i = (int64_t)g * 16 + li;
        const f64x4 V = column_spread<KX, true>(load_col<KX>(gc + g * 16, n), mp, n);
        if (i >= nt) continue;
        const f64x4 X = load_col<KX>(a.car + blk_at(i) * n, n) + V;
        store_col<KX>(a.car + blk_at(i) * n, X, n);
    }
    if constexpr (REV) {
        __syncthreads();
        if (wave == 0) {
            f64x4 X = zero4();
            if (len >= nh) {                 // the head's last step
                const f64x4 mk = load_col<KX>(static_cast<const R*>(a.m) + (sq.start + nh - 1) * n, n);
                X = mk;
                if (len > nh) {
                    const f64x4 Z = mm<KX>(load_op<KX>(mp, n, n), load_col<KX>(a.car + t0 * n, n),
                                           load_col<KX>(a.agg + t0 * n, n));
                    const f64x4 p = mm<KX>(load_op<KX>(a.F, n, n), mk, a.u ? load_col<KX>(a.u, n) : zero4());
                    X = mm<KX>(load_op<KX>(a.star + star_E(n, a.ny), n, n), Z - p, mk);
                }
            }
            for (int w = 0; w * q < nrun; ++w) {
                const f64x4 V = load_col<KX>(cb + w * 16, n);
                if (li == 0) store_col<KX>(cb + w * 16, X, n);
                X = mm<KX>(load_op<KX>(cm + w * kTile, 16, 16), X, V);
            }
        }
        __syncthreads();
    }
    if (i0 < i1) {
        f64x4 X = load_col<KX>(cb + wave * 16, n);
#pragma unroll 1
        for (int i = i0; i < i1; ++i) {
            const f64x4 op = load_op<KX>(runM + (int64_t)run_at(i) * n2, n, n);
            const f64x4 V = load_col<KX>(run_vec(a, a.runB, b, run_at(i)), n);
            if (li == 0) store_col<KX>(run_vec(a, a.runX, b, run_at(i)), X, n);
            X = mm<KX>(op, X, V);
        }
    }
}

// filtered means, and the chains and head runs of the smoother from zero,
// backwards; the rest of the smoothed head covariances
template <typename R, int KX, int KY>
__global__ __launch_bounds__(kWG) void k_st_filter_down(Args a, Grid g) {
    __shared__ double st[4][kStage];
    __shared__ double ag[4][16];
    const int nh = a.ctl[0];
    if (nh == 0) return;
    const int n = a.nx, m = a.ny, wave = threadIdx.x >> 6;
    int64_t blk = blockIdx.x;
    if (blk < g.heads) {
        int group, run;
        if (!head_wave(a, nh, blk, wave, group, run)) return;
        const Head h = head_of(a, nh, group);
        f64x4 rows[kRun], mk[kRun];
        const f64x4 X0 = load_col<KX>(run_vec(a, a.runX, h.b, run), n);
        run_filter<R, KX, KY, true>(a, h, run, X0, rows);
        if (!a.smooth) return;
#pragma unroll
        for (int v = 0; v < 4; ++v) mk[0][v] = double(R(X0[v]));
#pragma unroll
        for (int j = 1; j < kRun; ++j) mk[j] = rows[j - 1];
        const f64x4 Z = run_smoother<R, KX, false>(a, h, run, zero4(), mk);
        if (h.full > 0) store_col<KX>(run_vec(a, a.runB, h.b, run), Z, n);
        return;
    }
    blk -= g.heads;
    if (blk < g.extra) {
        const int i = (int)blk * 4 + wave;
        if (i < nh / kRun) head_fill<KX>(a, i, st[wave]);
        return;
    }
    blk -= g.extra;
    if (blk >= a.blk_off[a.B]) return;
    const Chain c = chain_of(a, nh, blk, wave);
    const R* y = static_cast<const R*>(a.y) + c.start * m;
    R* mo = static_cast<R*>(a.m) + c.start * n;
    const int64_t last = c.len - 1;
    const int L = 1 << a.pL;
    double* pre = a.pre + ((blk * 4 + wave) * 16 + lane_i()) * n;
    {
        const f64x4 PhiT = load_op<KX>(a.star + star_Phi(n, m), n, n), KT = load_op<KY>(a.star + star_K(n, m), n, m);
        const f64x4 cc = load_col<KX>(a.star + star_c(n, m), n);
        auto at = [&](int64_t k) { return load_col<KY>(y + (k < last ? k : last) * m, m); };
        f64x4 yy[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) yy[j] = at(c.k0 + j);
        const f64x4 M16 = load_op<KX>(a.mpF + (int64_t)4 * n * n, n, n);
        f64x4 V = load_col<KX>(a.car + blk * n, n);
        for (int s = 0; s < wave; ++s) V = mm<KX>(M16, V);
        f64x4 X = load_col<KX>(pre, n) + column_spread<KX, true>(V, a.mpF, n);
        for (int i = 0; i < L; i += 4) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f64x4 yk = yy[j];
                yy[j] = at(c.k0 + i + j + 4);
                X = mm<KX>(PhiT, X, mm<KY>(KT, yk, cc));
                if (c.k0 + i + j <= last) store_col<KX>(mo + (c.k0 + i + j) * n, X, n);
            }
        }
    }
    if (!a.smooth) return;
    const f64x4 FT = load_op<KX>(a.F, n, n), u = a.u ? load_col<KX>(a.u, n) : zero4();
    const f64x4 ET = load_op<KX>(a.star + star_E(n, m), n, n);
    f64x4 Z = zero4();
    auto at = [&](int64_t k) { return load_col<KX>(mo + (k < last ? k : last) * n, n); };
    f64x4 mm_[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) mm_[j] = at(c.k0 + L - 1 - j);
    for (int i = L - 1; i >= 0; i -= 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const f64x4 mk = mm_[j];
            const int64_t k = c.k0 + i - j, kn = k - 4;
            mm_[j] = at(kn > c.k0 ? kn : c.k0);
            const f64x4 Zn = mm<KX>(ET, Z - mm<KX>(FT, mk, u), mk);
#pragma unroll
            for (int v = 0; v < 4; ++v) Z[v] = k > last ? 0.0 : (k == last ? mk[v] : Zn[v]);
        }
    }
    Z = column_scan<KX, false>(Z, a.mpE, n);
    if (lane_i() == 0) store_col<KX>(ag[wave], Z, n);
    __syncthreads();
    const f64x4 M16 = load_op<KX>(a.mpE + (int64_t)4 * n * n, n, n);
    f64x4 V = zero4();
    for (int s = 3; s > wave; --s) V = mm<KX>(M16, V, load_col<KX>(ag[s], n));
    store_col<KX>(pre, shift<false, 1, KX>(Z) + column_spread<KX, false>(V, a.mpE, n), n);
    if (wave == 0) {
        V = mm<KX>(M16, V, load_col<KX>(ag[0], n));
        if (lane_i() == 0) store_col<KX>(a.agg + blk * n, V, n);
    }
}

// smoothed means; Ps
template <typename R, int KX>
__global__ __launch_bounds__(kWG) void k_st_smoother_down(Args a, Grid g) {
    __shared__ double st[4][kStage];
    __shared__ __align__(16) R row[256];
    const int nh = a.ctl[0];
    if (nh == 0) return;
    const int n = a.nx, m = a.ny, wave = threadIdx.x >> 6;
    int64_t blk = blockIdx.x;
    if (blk < g.heads) {
        int group, run;
        if (!head_wave(a, nh, blk, wave, group, run)) return;
        const Head h = head_of(a, nh, group);
        const R* mi = static_cast<const R*>(a.m) + h.start * n;
        f64x4 mk[kRun];
#pragma unroll
        for (int j = 0; j < kRun; ++j) {
            const int k = run * kRun - 1 + j;
            mk[j] = k >= 0 && k < h.len ? load_col<KX>(mi + (int64_t)k * n, n) : zero4();
        }
        const f64x4 Z = load_col<KX>(run_vec(a, a.runX, h.b, run), n);
        if ((run + 1) * kRun == nh && h.len == nh)
            store_col<KX>(static_cast<R*>(a.ms) + (h.start + nh - 1) * n, Z, n);
        run_smoother<R, KX, true>(a, h, run, Z, mk);
        return;
    }
    blk -= g.heads;
    if (blk < g.extra) {          // short sequences
        const int b = (int)blk * 4 + wave;
        if (b < a.B) short_head<R, KX>(a, nh, b, st[wave]);
        return;
    }
    blk -= g.extra;
    if (blk >= g.blocks) {
        write_rows<R, true>(a, nh, blk - g.blocks, gridDim.x - g.heads - g.extra - g.blocks, row);
        return;
    }
    if (blk >= a.blk_off[a.B]) return;
    const Chain c = chain_of(a, nh, blk, wave);
    const R* mi = static_cast<const R*>(a.m) + c.start * n;
    R* mo = static_cast<R*>(a.ms) + c.start * n;
    const int64_t last = c.len - 1;
    const int L = 1 << a.pL;
    auto at = [&](int64_t k) { return load_col<KX>(mi + (k < last ? k : last) * n, n); };
    f64x4 mm_[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) mm_[j] = at(c.k0 + L - 1 - j);
    const f64x4 FT = load_op<KX>(a.F, n, n), u = a.u ? load_col<KX>(a.u, n) : zero4();
    const f64x4 ET = load_op<KX>(a.star + star_E(n, m), n, n);
    const f64x4 M16 = load_op<KX>(a.mpE + (int64_t)4 * n * n, n, n);
    f64x4 V = load_col<KX>(a.car + blk * n, n);
    for (int s = 3; s > wave; --s) V = mm<KX>(M16, V);
    f64x4 Z = load_col<KX>(a.pre + ((blk * 4 + wave) * 16 + lane_i()) * n, n) + column_spread<KX, false>(V, a.mpE, n);
    for (int i = L - 1; i >= 0; i -= 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const f64x4 mk = mm_[j];
            const int64_t k = c.k0 + i - j, kn = k - 4;
            mm_[j] = at(kn > c.k0 ? kn : c.k0);
            const f64x4 Zn = mm<KX>(ET, Z - mm<KX>(FT, mk, u), mk);
            if (k <= last) {
                Z = k == last ? mk : Zn;
                store_col<KX>(mo + k * n, Z, n);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
template <typename R, int KX, int KY>
hipError_t run(const Args& a, hipStream_t s) {
    const int writers = 1024;
    const int64_t heads = ((int64_t)((a.B + 15) / 16) * (a.N / kRun) + 3) / 4;
    prof_begin("k_st_double", s);
    hipLaunchKernelGGL((k_st_double<KX, KY>), dim3(1), dim3(64), 0, s, a);
    prof_end(s);
    prof_begin("k_st_tables", s);
    hipLaunchKernelGGL((k_st_tables<KX, KY>), dim3(2 + (a.smooth ? 2 : 1) * (a.N / kRun)), dim3(64), 0, s, a);
    prof_end(s);
    Grid g{heads, 0, a.max_blocks};
    prof_begin("k_st_filter_reduce", s);
    hipLaunchKernelGGL((k_st_filter_reduce<R, KX, KY>), dim3((unsigned)(g.heads + g.blocks + writers)), dim3(kWG), 0, s, a, g);
    prof_end(s);
    prof_begin("k_st_filter_top", s);
    hipLaunchKernelGGL((k_st_top<R, KX, false>), dim3(a.B + (a.smooth ? 1 : 0)), dim3(64 * kTopWaves), 0, s, a);
    prof_end(s);
    g.extra = a.smooth ? (a.N / kRun + 3) / 4 : 0;
    prof_begin("k_st_filter_down", s);
    hipLaunchKernelGGL((k_st_filter_down<R, KX, KY>), dim3((unsigned)(g.heads + g.extra + g.blocks)), dim3(kWG), 0, s, a, g);
    prof_end(s);
    if (a.smooth) {
        prof_begin("k_st_smoother_top", s);
        hipLaunchKernelGGL((k_st_top<R, KX, true>), dim3(a.B), dim3(64 * kTopWaves), 0, s, a);
        prof_end(s);
        g.extra = (a.B + 3) / 4;
        prof_begin("k_st_smoother_down", s);
        hipLaunchKernelGGL((k_st_smoother_down<R, KX>), dim3((unsigned)(g.heads + g.extra + g.blocks + writers)), dim3(kWG),
                           0, s, a, g);
        prof_end(s);
    }
    return hipGetLastError();
}

template <typename R, int KX>
hipError_t run_ky(const Args& a, hipStream_t s) {
    switch (slices(a.ny)) {
        case 1: return run<R, KX, 1>(a, s);
        case 2: return run<R, KX, 2>(a, s);
        default: return run<R, KX, 4>(a, s);
    }
}
template <typename R>
hipError_t run_kx(const Args& a, hipStream_t s) {
    switch (slices(a.nx)) {
        case 1: return run_ky<R, 1>(a, s);
        case 2: return run_ky<R, 2>(a, s);
        default: return run_ky<R, 4>(a, s);
    }
}

}  // namespace

// Sizes alone decide.  The setup is a chain of latencies (nx = 4: 55 us, nx = 16:
// 100 us) whatever the length, the general scan's arithmetic grows with T nx^3.
// Filter + smoother, us, general and here, of models that settle in 256 steps (CV at
// 10 Hz), nx = 3: constant acceleration, 512:
//   nx = 4: FP64  T = 98304 115, 106; 2^17 120, 107; 2^18 141, 117; 2^20 243, 181
//           mixed T = 196608 111, 110; 2^18 122, 114; 393216 155, 124; 2^20 191, 162 (its
//           general kernels multiply in FP32)
//   nx = 3: FP64  T = 233017 124, 121; 2^18 134, 122; 2^20 368, 180
//           mixed T = 466101 140, 142; 2^19 147, 148; 2^20 274, 181
//   nx <= 2: 123 general, 153 here at T = 2^20
//   nx = 6: T = 8192 268, 145; nx = 16: 319, 242; nx = 24: 3163, 498; nx = 64: 59867, 1778
// A model that does not settle in the tables' steps costs the doubling and the idle
// launches on top: 17 to 23 us at nx <= 4, 25 at nx = 6, 55 to 60 at nx = 16 (70 the
// filter alone), 130 at nx = 24, 500 at nx = 64.
// Packed sequences: the tables hold a quarter of the mean length at most.  At a mean of
// 1024 that is 256 steps; at 512, 128 steps serve only the faster models (64 sequences
// of nx = 16, settling in 128: 563 general, 243 here; of one that does not, 8 % lost).
constexpr int64_t kMinSteps = 8192, kMinMean = 1024;
constexpr int64_t kMinWorkF64 = 6 << 20, kMinWorkF32 = 12 << 20;     // T nx^3, nx <= 4

bool applies(int nx, int ny, int32_t B, int64_t total, bool mixed) {
    if (ny > (nx + 15) / 16 * 16 || total < kMinSteps || total / B < kMinMean) return false;
    return nx > 4 || (nx > 2 && total * nx * nx * nx >= (mixed ? kMinWorkF32 : kMinWorkF64));
}

bool layout(Args& a, char* base, size_t bytes) {
    const int64_t n = a.nx, m = a.ny, n2 = n * n;
    // at least 16 steps a chain, at most 32768 chains (2048 waves)
    const bool large = a.nx > 16;        // 16 chains a workgroup, at most 16384
    a.pL = 4;
    while ((a.total >> a.pL) > (large ? 16384 : 32768)) ++a.pL;
    const int64_t chains = large ? 16 : kBlockChains;
    a.max_blocks = a.total / (chains << a.pL) + a.B;
    for (a.N = 1024; a.N >= 64; a.N /= 2) {
        if (a.N > a.total / a.B / 4) continue;
        char* p = base;
        auto take = [&](int64_t words) {
            double* q = reinterpret_cast<double*>(p);
            p += ((size_t)words * sizeof(double) + 255) & ~size_t(255);
            return q;
        };
        int levels = 1;
        while ((1 << (levels - 1)) < a.N) ++levels;
        const int64_t runs = a.N / kRun;
        a.blk_off = reinterpret_cast<int64_t*>(take(a.B + 1));
        a.star = take(star_words(a.nx, a.ny));
        a.powF = take(levels * 3 * n2);
        a.powE = take(levels * 2 * n2);
        a.mpF = take(kPowers * n2);
        a.mpE = take(kPowers * n2);
        a.tP = take(a.N * n2);
        a.tPhi = take(a.N * n2);
        a.tK = take(a.N * n * m);
        a.tc = take(a.N * n);
        a.tE = take(a.N * n2);
        a.tL = take(a.N * n2);
        a.tHead = take(a.N * n2);
        a.tTail = take(a.N * n2);
        a.runPhi = take(runs * n2);
        a.runE = take(runs * n2);
        a.runL = take(runs * n2);
        a.runC = large ? nullptr : take(runs * n2);
        for (int i = 0; i < 2; ++i) {
            a.scanE[i] = large ? take(runs * n2) : nullptr;
            a.scanL[i] = large ? take(runs * n2) : nullptr;
        }
        a.pre = take(a.max_blocks * chains * n);
        a.agg = take(a.max_blocks * n);
        a.car = take(a.max_blocks * n);
        a.runB = take(a.B * runs * n);
        a.runX = take(a.B * runs * n);
        if ((size_t)(p - base) <= bytes) return true;
    }
    return false;
}

hipError_t launch(Args a, bool mixed, hipStream_t s) {
    if (a.nx > 16) return launch_large(a, mixed, s);
    return mixed ? run_kx<float>(a, s) : run_kx<double>(a, s);
}

}  // namespace steady
}  // namespace pks
