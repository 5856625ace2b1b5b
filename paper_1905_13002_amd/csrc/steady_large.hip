// steady_large.hip -- filter and smoother of a time-invariant model with
// settled covariances (see steady.hpp), 16 < nx <= 64 and ny <= the next
// multiple of 16 above nx.
//
// Setup: a workgroup of NT x NT waves holds each matrix as one 16 x 16 register
// tile a wave (NT = 2, 3, 4); products exchange tiles through LDS and run on
// v_mfma_f64_16x16x4f64, inverses are Gauss-Jordan by blocks of 16 (the
// diagonal block in one wave's registers, the rest as products).  The
// formulas are those of steady.hip, matrix for matrix.
// Means: a workgroup of NT waves steps 16 chains, wave t the rows 16 t .. of
// their states, which it publishes in LDS for the next step's product.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "steady_ops.hpp"

namespace pks {
namespace steady {

namespace {

constexpr int kLargePowers = 9;       // L .. 256 L

// ---------------------------------------------------------------------------
// matrices spread over the waves of a workgroup: wave (r, c) holds block (r, c)
// ---------------------------------------------------------------------------
template <int NT>
struct Eng {
    static constexpr int kTiles = NT * NT;
    static constexpr int kLds = (2 * kTiles + 1) * kTile + 8;      // doubles
    double *b0, *b1, *db;
    int* flag;
    int r, c, w, n, m;

    __device__ __forceinline__ Eng(double* lds, const Args& a) {
        b0 = lds;
        b1 = b0 + kTiles * kTile;
        db = b1 + kTiles * kTile;
        flag = reinterpret_cast<int*>(db + kTile);
        w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        r = w / NT;
        c = w % NT;
        n = a.nx;
        m = a.ny;
    }
    // block (r, c) of a rows x cols matrix in memory, and of its transpose
    __device__ __forceinline__ f64x4 ld(const double* X, int rows, int cols) const {
        return load_tile(X + (int64_t)16 * r * cols + 16 * c, rows - 16 * r, cols - 16 * c, cols);
    }
    __device__ __forceinline__ f64x4 ldt(const double* X, int rows, int cols) const {
        return load_tile_t(X + (int64_t)16 * c * cols + 16 * r, rows - 16 * c, cols - 16 * r, cols);
    }
    template <typename T>
    __device__ __forceinline__ void st(T* X, const f64x4& x, int rows, int cols) const {
        const int li = 16 * c + lane_i(), lk = 16 * r + lane_k();
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (lk + 4 * v < rows && li < cols) X[(int64_t)(lk + 4 * v) * cols + li] = T(x[v]);
    }
    __device__ __forceinline__ f64x4 id() const { return r == c ? eye() : zero4(); }
    // the identity beyond k on the diagonal (and zero there: `clear`)
    __device__ __forceinline__ f64x4 pad(f64x4 x, int k, double value = 1.0) const {
        const int li = lane_i(), lk = lane_k();
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (r == c && 4 * v + lk == li && 16 * r + li >= k) x[v] = value;
        return x;
    }
    // tile of the transpose of a staged tile
    static __device__ __forceinline__ f64x4 get_t(const double* p) {
        const int li = lane_i(), lk = lane_k();
        f64x4 t;
#pragma unroll
        for (int v = 0; v < 4; ++v) t[v] = p[((li & 3) * 16 + 4 * v + lk) * 4 + (li >> 2)];
        return t;
    }
    // X^T Y + acc
    __device__ __forceinline__ f64x4 xty(const f64x4& x, const f64x4& y, f64x4 acc) const {
        put_tile(b0 + w * kTile, x);
        put_tile(b1 + w * kTile, y);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NT; ++k) acc = mm(get_tile(b0 + (k * NT + r) * kTile), get_tile(b1 + (k * NT + c) * kTile), acc);
        __syncthreads();
        return acc;
    }
    __device__ __forceinline__ f64x4 xty(const f64x4& x, const f64x4& y) const { return xty(x, y, zero4()); }
    __device__ __forceinline__ f64x4 tr(const f64x4& x) const {
        put_tile(b0 + w * kTile, x);
        __syncthreads();
        const f64x4 t = get_t(b0 + (c * NT + r) * kTile);
        __syncthreads();
        return t;
    }
    __device__ __forceinline__ f64x4 symt(const f64x4& x, const f64x4& add) const { return sym(x, tr(x), add); }
    __device__ __forceinline__ bool any(bool x) const {
        if (threadIdx.x == 0) *flag = 0;
        __syncthreads();
        if (x) *flag = 1;
        __syncthreads();
        const bool t = *flag != 0;
        __syncthreads();
        return t;
    }
    // inverse by Gauss-Jordan over blocks of 16, without pivoting (rows beyond
    // the matrix hold the identity); `ok` is cleared by a zero (SPD: not
    // positive) or non-finite pivot
    template <bool SPD>
    __device__ __forceinline__ f64x4 inv(f64x4 a, bool& ok) const {
        bool good = true;
#pragma unroll 1
        for (int kb = 0; kb < NT; ++kb) {
            if (r == kb || c == kb) put_tile(b0 + w * kTile, a);
            if (r == kb && c == kb) {
                a = inv_np<16, SPD>(a, good);
                put_tile(db, a);
            }
            __syncthreads();
            if (r == kb && c != kb) {
                a = mm(get_t(db), a);
                put_tile(b1 + c * kTile, a);
            }
            __syncthreads();
            if (r != kb) {
                const f64x4 left = -get_t(b0 + (r * NT + kb) * kTile);
                a = c == kb ? mm(left, get_tile(db)) : mm(left, get_tile(b1 + c * kTile), a);
            }
            __syncthreads();
        }
        ok = ok && !any(!good);
        return a;
    }
    // S^-1 X given the inverse Si of the symmetric S, refined once (as in steady.hip)
    __device__ __forceinline__ f64x4 solve(const f64x4& S, const f64x4& Si, const f64x4& X) const {
        const f64x4 q = xty(Si, X);
        return xty(Si, X - xty(S, q), q);
    }
    // E L E^T + add, E by its transpose
    __device__ __forceinline__ f64x4 ele(const f64x4& ET, const f64x4& L, const f64x4& add) const {
        return symt(xty(xty(L, ET), ET), add);
    }
    // (negligible, meets: as in steady.hip)
    __device__ __forceinline__ bool negligible(const f64x4& AT, const f64x4& P, const f64x4& C, double f) const {
        const f64x4 R = xty(AT, xty(P, AT));
        return !any(r == c && !diagonal_below(R, C, f, n - 16 * r));
    }
    __device__ __forceinline__ bool meets(const f64x4& x, const f64x4& y) const {
        const f64x4 d = r == c ? diagonal(y) : zero4(), di = xty(d, ones()), dj = xty(ones(), d);
        return !any(!steady::meets(x, y, di, dj));
    }
    // (M^T)^-1 for M = I + C J: refined where the residual is not rounding; `ok` is
    // cleared where it is not small
    __device__ __forceinline__ f64x4 inv_ijc(const f64x4& C, const f64x4& J, bool& ok) const {
        const f64x4 I = id();
        const f64x4 N = inv<false>(xty(J, C, I), ok);
        const f64x4 R = xty(xty(C, J, I), N);
        double dev = 0.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) dev = fmax(dev, fabs(R[v] - I[v]));
        if (!any(!(dev <= kExact))) return N;
        ok = ok && !any(!(dev <= kSmall));
        return xty(tr(N), I - R, N);
    }
};

// A word that other workgroups of the launch may clear meanwhile: the same value in
// every wave of this one, which meet at barriers behind it
__device__ __forceinline__ int read_once(const int* p) {
    __shared__ int v;
    if (threadIdx.x == 0) v = *p;
    __syncthreads();
    return v;
}

template <int NT>
struct ModelL {
    f64x4 F, FT, Q, HT, R;
};
template <int NT>
__device__ __forceinline__ ModelL<NT> load_model(const Eng<NT>& e, const Args& a) {
    ModelL<NT> x;
    x.F = e.ld(a.F, e.n, e.n);
    x.FT = e.ldt(a.F, e.n, e.n);
    x.Q = e.pad(e.ld(a.Q, e.n, e.n), e.n);
    x.HT = e.ldt(a.H, e.m, e.n);
    x.R = e.pad(e.ld(a.R, e.m, e.m), e.m);
    return x;
}
template <int NT>
__device__ __forceinline__ void predict(const Eng<NT>& e, const ModelL<NT>& x, const f64x4& P, f64x4& FP, f64x4& Pm) {
    FP = e.xty(x.FT, P);
    Pm = e.symt(e.xty(x.FT, e.tr(FP), x.Q), zero4());
}
template <int NT>
__device__ __forceinline__ void update(const Eng<NT>& e, const ModelL<NT>& x, const f64x4& Pm, bool& ok, f64x4& P, f64x4& Kt,
                                       f64x4& Phi) {
    const f64x4 HP = e.xty(x.HT, Pm);
    const f64x4 S = e.symt(e.xty(x.HT, e.tr(HP), x.R), zero4());
    Kt = e.solve(S, e.template inv<true>(S, ok), HP);
    const f64x4 nKt = -Kt;
    P = e.pad(e.symt(e.xty(nKt, HP, Pm), zero4()), e.n, 0.0);
    Phi = e.xty(nKt, e.xty(x.HT, x.F), x.F);
}
template <int NT>
__device__ __forceinline__ void smooth_elem(const Eng<NT>& e, const f64x4& P, const f64x4& FP, const f64x4& Pm, bool& ok,
                                            f64x4& ET, f64x4& L) {
    ET = e.solve(Pm, e.template inv<true>(Pm, ok), FP);
    const f64x4 EFP = e.xty(ET, FP), EFPt = e.tr(EFP);
#pragma unroll
    for (int v = 0; v < 4; ++v) L[v] = P[v] - 0.5 * (EFP[v] + EFPt[v]);
}
// c = u - K (H u + d), K by the staged tiles of K^T (in e.b0)
template <int NT>
__device__ __forceinline__ void gain_offset(const Eng<NT>& e, const Args& a, const f64x4& Kt, double* out) {
    double* hu = e.b1;
    put_tile(e.b0 + e.w * kTile, Kt);
    for (int q = threadIdx.x; q < e.m; q += blockDim.x) {
        double s = a.d ? a.d[q] : 0.0;
        if (a.u)
            for (int l = 0; l < e.n; ++l) s = fma(a.H[(int64_t)q * e.n + l], a.u[l], s);
        hu[q] = s;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < e.n; i += blockDim.x) {
        double s = a.u ? a.u[i] : 0.0;
        for (int q = 0; q < e.m; ++q) {
            // K^T(q, i): lane (q % 4, i % 16), component (q % 16) / 4 of block (q / 16, i / 16)
            const double* t = e.b0 + ((q >> 4) * NT + (i >> 4)) * kTile;
            s = fma(-t[((q & 3) * 16 + (i & 15)) * 4 + ((q & 15) >> 2)], hu[q], s);
        }
        out[i] = s;
    }
    __syncthreads();
}

// The smoother alone.  Whether it is worth the setup (0.3 ms at nx = 24): the last
// two filtered covariances of the longest sequence are the same (ctl[3] = 0).
// 40 sequences of 100 to 2000 steps, nx = 24, mixed: 0.5 ms, of which the
// comparison below is 30 us; by the general kernels 4.0 ms.
template <typename R>
__global__ __launch_bounds__(256) void k_stl_probe(Args a) {
    __shared__ int64_t best[256];
    const int t = threadIdx.x;
    int64_t len = a.total, end = a.total;
    if (a.offsets) {
        len = 0;
        for (int b = t; b < a.B; b += 256) {
            const int64_t s = a.offsets[b], e = a.offsets[b + 1];
            if (e - s > len) {
                len = e - s;
                end = e;
            }
        }
        best[t] = len;
        __syncthreads();
        int w = 0;
        for (int i = 1; i < 256; ++i)
            if (best[i] > best[w]) w = i;
        __syncthreads();
        if (t == w) best[0] = end;
        __syncthreads();
        end = best[0];
    }
    const int n2 = a.nx * a.nx;
    const R* P = static_cast<const R*>(a.P) + (end - 1) * n2;
    bool differs = false;
    for (int i = t; i < n2; i += 256) differs |= !(P[i] == P[i - n2]);
    differs = __syncthreads_or(differs) != 0;
    if (t == 0) a.ctl[3] = differs ? 1 : 0;
}
// and, with the tables there, whether every covariance is the filter's
template <typename R>
__global__ __launch_bounds__(256) void k_stl_check(Args a) {
    extern __shared__ __align__(16) double dyn[];
    const int nh = read_once(a.ctl);
    if (nh == 0) return;
    if (rows_differ<R>(a, nh, blockIdx.x, gridDim.x, reinterpret_cast<R*>(dyn))) a.ctl[0] = 0;
}


// ---------------------------------------------------------------------------
// Doubling: one workgroup, bound by the chain of about log2 n combines
// ---------------------------------------------------------------------------
template <int NT>
__global__ __launch_bounds__(64 * NT * NT) void k_stl_double(Args a) {
    extern __shared__ __align__(16) double lds[];
    const Eng<NT> e(lds, a);
    const int n = a.nx, n2 = n * n, m = a.ny;
    if (threadIdx.x == 0) {
        if (a.reset || a.status[1] != kStatusMagic) {
            a.status[0] = kStatusOk;
            a.status[1] = kStatusMagic;
        }
        a.ctl[0] = 0;
    }
    if (a.given && a.ctl[3] != 0) return;
    const ModelL<NT> x = load_model(e, a);
    bool ok = true;
    f64x4 A, C, J;
    {
        const f64x4 Q = e.ld(a.Q, n, n);
        const f64x4 T1 = e.xty(x.HT, Q);
        const f64x4 S = e.symt(e.xty(e.tr(T1), x.HT, x.R), zero4());
        const f64x4 Si = e.template inv<true>(S, ok);
        const f64x4 nKt = -e.xty(Si, T1), G = e.xty(x.HT, x.F);
        J = e.symt(e.xty(G, e.xty(Si, G)), zero4());
        A = e.xty(nKt, G, x.F);
        C = e.symt(e.xty(nKt, T1, Q), zero4());
    }
    e.st(a.powF, A, n, n);
    e.st(a.powF + n2, C, n, n);
    e.st(a.powF + 2 * n2, J, n, n);
    const f64x4 P0 = e.ld(a.P0, n, n);
    int lf = 0, le = 0;
    bool settled = false;
    f64x4 AT = e.tr(A);
#pragma unroll 1
    for (int l = 1; (1 << l) <= a.N && ok; ++l) {
        const f64x4 N = e.inv_ijc(C, J, ok);
        const f64x4 X1 = e.xty(N, A), X3 = e.xty(N, C), JA = e.xty(J, A);
        A = e.xty(AT, X1);
        C = e.symt(e.xty(AT, e.xty(X3, AT)), C);
        J = e.symt(e.xty(X1, JA), J);
        AT = e.tr(A);
        double* rec = a.powF + (int64_t)l * 3 * n2;
        e.st(rec, A, n, n);
        e.st(rec + n2, C, n, n);
        e.st(rec + 2 * n2, J, n, n);
        lf = l;
        if ((1 << l) >= kRun && e.negligible(AT, P0 + C, C, kTiny)) {
            settled = true;
            break;
        }
    }
    if (!(settled && ok)) return;
    const f64x4 P = C;
    f64x4 FP, Pm, Kt, Phi, ET, L, Pn;
    predict(e, x, P, FP, Pm);
    smooth_elem(e, P, FP, Pm, ok, ET, L);
    update(e, x, Pm, ok, Pn, Kt, Phi);
    e.st(a.star + star_P(n, m), P, n, n);
    e.st(a.star + star_Phi(n, m), Phi, n, n);
    e.st(a.star + star_K(n, m), e.tr(Kt), n, m);
    gain_offset(e, a, Kt, a.star + star_c(n, m));
    e.st(a.star + star_E(n, m), e.tr(ET), n, n);
    e.st(a.star + star_L(n, m), L, n, n);
    settled = false;
#pragma unroll 1
    for (int l = 0; (1 << l) <= a.N && ok; ++l) {
        f64x4 E = e.tr(ET);
        if (l > 0) {
            L = e.ele(ET, L, L);
            ET = e.xty(E, ET);                       // (E E)^T
            E = e.tr(ET);
        }
        e.st(a.powE + (int64_t)l * 2 * n2, E, n, n);
        e.st(a.powE + (int64_t)l * 2 * n2 + n2, L, n, n);
        le = l;
        if ((1 << l) >= kRun && e.negligible(ET, P, L, kTiny)) {
            settled = true;
            break;
        }
    }
    if (!(settled && ok)) return;
    e.st(a.star + star_Ps(n, m), L, n, n);
    // the tiles of every sequence: 16 chains of L steps beyond the head
    if (threadIdx.x >= 64) return;
    const int lane = threadIdx.x, nh = 1 << (lf > le ? lf : le);
    const int64_t per = (int64_t)16 << a.pL;
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

// head and tail tables and the powers of Phi and E (a workgroup per run)
template <int NT>
__global__ __launch_bounds__(64 * NT * NT) void k_stl_tables(Args a) {
    extern __shared__ __align__(16) double lds[];
    const int nh = read_once(a.ctl);
    if (nh == 0) return;
    const Eng<NT> e(lds, a);
    const int nrun = nh / kRun, n = a.nx, n2 = n * n, m = a.ny;
    const int lf = a.ctl[1], le = a.ctl[2];
    int blk = blockIdx.x;
    if (blk < 2) {
        if (blk == 1 && !a.smooth) return;
        const double* src = a.star + (blk == 0 ? star_Phi(n, m) : star_E(n, m));
        double* out = blk == 0 ? a.mpF : a.mpE;
        f64x4 M = e.ld(src, n, n);
#pragma unroll 1
        for (int p = 0; p < a.pL + kLargePowers; ++p) {
            if (p >= a.pL) e.st(out + (int64_t)(p - a.pL) * n2, M, n, n);
            M = e.xty(e.tr(M), M);
        }
        return;
    }
    blk -= 2;
    if (blk >= (a.smooth ? 2 : 1) * nrun) return;
    bool ok = true;
    if (blk >= nrun) {                       // tail
        const int j0 = (blk - nrun) * kRun;
        f64x4 Ps;
        if (j0 >> le) {
            Ps = e.ld(a.star + star_Ps(n, m), n, n);
        } else {
            Ps = e.ld(a.star + star_P(n, m), n, n);
#pragma unroll 1
            for (int l = 0; (j0 >> l) != 0; ++l)
                if ((j0 >> l) & 1) {
                    const double* rec = a.powE + (int64_t)l * 2 * n2;
                    Ps = e.ele(e.ldt(rec, n, n), Ps, e.ld(rec + n2, n, n));
                }
        }
        const f64x4 ET = e.ldt(a.star + star_E(n, m), n, n), L = e.ld(a.star + star_L(n, m), n, n);
#pragma unroll 1
        for (int j = j0; j < j0 + kRun; ++j) {
            e.st(a.tTail + (int64_t)j * n2, Ps, n, n);
            Ps = e.ele(ET, Ps, L);
        }
        if (j0 + kRun == 1 << le && !e.meets(Ps, e.ld(a.star + star_Ps(n, m), n, n)) && threadIdx.x == 0)
            atomicExch(&a.ctl[0], 0);
        return;
    }
    const int k0 = blk * kRun;
    const ModelL<NT> x = load_model(e, a);
    f64x4 P = e.ld(a.P0, n, n);
    const f64x4 Pstar = e.ld(a.star + star_P(n, m), n, n);
    const f64x4 AnT = e.ldt(a.powF + (int64_t)lf * 3 * n2, n, n);       // of the steps that it takes to settle
    if (k0 >> lf) {
        P = Pstar;
    } else {
#pragma unroll 1
        for (int l = 0; (k0 >> l) != 0; ++l)
            if ((k0 >> l) & 1) {
                const double* rec = a.powF + (int64_t)l * 3 * n2;
                const f64x4 AT = e.ldt(rec, n, n);
                const f64x4 X3 = e.xty(e.inv_ijc(P, e.ld(rec + 2 * n2, n, n), ok), P);
                P = e.symt(e.xty(AT, e.xty(X3, AT)), e.ld(rec + n2, n, n));
            }
    }
    f64x4 EaT = e.id(), La = zero4(), Pa = e.id();
#pragma unroll 1
    for (int k = k0; k < k0 + kRun; ++k) {
        f64x4 FP, Pm, Kt, Phi;
        predict(e, x, P, FP, Pm);
        if (a.smooth && k > 0) {             // of step k - 1, whose covariance P is
            f64x4 ET, L;
            smooth_elem(e, P, FP, Pm, ok, ET, L);
            const f64x4 E = e.tr(ET);
            e.st(a.tE + (int64_t)(k - 1) * n2, E, n, n);
            e.st(a.tL + (int64_t)(k - 1) * n2, L, n, n);
            La = e.ele(EaT, L, La);
            EaT = e.xty(E, EaT);             // (E_a E)^T
        }
        update(e, x, Pm, ok, P, Kt, Phi);
        ok = e.negligible(AnT, P, Pstar, kSpare * kTiny) && ok;
        Pa = e.xty(e.tr(Phi), Pa);
        e.st(a.tP + (int64_t)k * n2, P, n, n);
        e.st(a.tPhi + (int64_t)k * n2, Phi, n, n);
        e.st(a.tK + (int64_t)k * n * m, e.tr(Kt), n, m);
        gain_offset(e, a, Kt, a.tc + (int64_t)k * n);
    }
    e.st(a.runPhi + (int64_t)blk * n2, Pa, n, n);
    if (a.smooth) {
        e.st(a.runE + (int64_t)blk * n2, e.tr(EaT), n, n);
        e.st(a.runL + (int64_t)blk * n2, La, n, n);
        if (k0 + kRun == nh) {               // E of the head's last step, whose covariance has settled
            e.st(a.tE + (int64_t)(nh - 1) * n2, e.ld(a.star + star_E(n, m), n, n), n, n);
            e.st(a.tL + (int64_t)(nh - 1) * n2, e.ld(a.star + star_L(n, m), n, n), n, n);
        }
    }
    if (k0 + kRun == 1 << lf) ok = e.meets(P, Pstar) && ok;
    if (!ok && threadIdx.x == 0) atomicExch(&a.ctl[0], 0);
}

// Smoothed covariances of the head: suffix scan of the runs' smoothing
// elements, one doubling of the distance a launch (out[i] = in[i] (x) in[i + d])
template <int NT>
__global__ __launch_bounds__(64 * NT * NT) void k_stl_head_scan(Args a, const double* inE, const double* inL, double* outE,
                                                               double* outL, int d) {
    extern __shared__ __align__(16) double lds[];
    const int nh = a.ctl[0], i = blockIdx.x;
    if (i >= nh / kRun) return;
    const Eng<NT> e(lds, a);
    const int n = a.nx, n2 = n * n;
    inE += (int64_t)i * n2;
    inL += (int64_t)i * n2;
    f64x4 E = e.ld(inE, n, n), L = e.ld(inL, n, n);
    if (i + d < nh / kRun) {
        const f64x4 ET = e.ldt(inE, n, n);
        L = e.ele(ET, e.ld(inL + (int64_t)d * n2, n, n), L);
        E = e.xty(ET, e.ld(inE + (int64_t)d * n2, n, n));
    }
    e.st(outE + (int64_t)i * n2, E, n, n);
    e.st(outL + (int64_t)i * n2, L, n, n);
}
// and the rows: run i from the settled covariance through everything behind it
template <int NT>
__global__ __launch_bounds__(64 * NT * NT) void k_stl_head_fill(Args a, const double* sE, const double* sL) {
    extern __shared__ __align__(16) double lds[];
    const int nh = a.ctl[0], i = blockIdx.x;
    if (i >= nh / kRun) return;
    const Eng<NT> e(lds, a);
    const int n = a.nx, n2 = n * n;
    f64x4 Ps = e.ld(a.star + star_Ps(n, a.ny), n, n);
    if (i + 1 < nh / kRun) Ps = e.ele(e.ldt(sE + (int64_t)(i + 1) * n2, n, n), Ps, e.ld(sL + (int64_t)(i + 1) * n2, n, n));
    int k = i * kRun + kRun - 1;
    e.st(a.tHead + (int64_t)k * n2, Ps, n, n);
    for (; k > i * kRun; --k) {
        Ps = e.ele(e.ldt(a.tE + (int64_t)(k - 1) * n2, n, n), Ps, e.ld(a.tL + (int64_t)(k - 1) * n2, n, n));
        e.st(a.tHead + (int64_t)(k - 1) * n2, Ps, n, n);
    }
}
// a sequence shorter than 2 n: its head folded from its own last covariances, a
// workgroup for the rows of each run, which the elements of the runs behind it
// reach in a step each (step by step, one workgroup a sequence: 204 us for 40
// sequences of nx = 24, a head of 128; so 55)
template <typename R, int NT>
__global__ __launch_bounds__(64 * NT * NT) void k_stl_short_head(Args a) {
    extern __shared__ __align__(16) double lds[];
    const int nh = a.ctl[0], run = blockIdx.y;
    if (nh == 0 || run >= nh / kRun) return;
    const SeqR q = seq_of(a, blockIdx.x);
    const int64_t len = q.end - q.start;
    if (len >= 2 * nh || len < 1) return;
    int k = (int)(len < nh ? len : nh) - 1;          // the step that Ps is of
    const int last = k / kRun;
    if (run > last) return;
    const Eng<NT> e(lds, a);
    const int n = a.nx, n2 = n * n;
    R* out = static_cast<R*>(a.Ps) + q.start * n2;
    f64x4 Ps = e.ld(len < nh ? a.tP + (int64_t)k * n2 : a.tTail + (len - nh) * n2, n, n);
    auto back = [&](const double* E, const double* L) { Ps = e.ele(e.ldt(E, n, n), Ps, e.ld(L, n, n)); };
    if (run < last) {
        for (; k >= last * kRun; --k) back(a.tE + (int64_t)(k - 1) * n2, a.tL + (int64_t)(k - 1) * n2);
        for (int r = last - 1; r > run; --r) back(a.runE + (int64_t)r * n2, a.runL + (int64_t)r * n2);
        k = run * kRun + kRun - 1;
    }
    if (run < last || len < nh) e.st(out + (int64_t)k * n2, Ps, n, n);
    for (; k > run * kRun; --k) {
        back(a.tE + (int64_t)(k - 1) * n2, a.tL + (int64_t)(k - 1) * n2);
        e.st(out + (int64_t)(k - 1) * n2, Ps, n, n);
    }
}

// ---------------------------------------------------------------------------
// means
// ---------------------------------------------------------------------------
// wave t's rows of the 16 columns, published for every wave
template <int NT>
struct Rows {
    f64x4 (*buf)[NT][64];      // [2]
    int ph = 0, t;
    __device__ __forceinline__ explicit Rows(f64x4 (*b)[NT][64]) : buf(b), t(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {}
    __device__ __forceinline__ void share(const f64x4& own, f64x4 (&all)[NT]) {
        buf[ph][t][threadIdx.x & 63] = own;
        __syncthreads();
#pragma unroll
        for (int s = 0; s < NT; ++s) all[s] = buf[ph][s][threadIdx.x & 63];
        ph ^= 1;
    }
};
// wave t's rows of a matrix as left operand
template <int NT>
struct Op {
    f64x4 f[NT];
};
template <int NT>
__device__ __forceinline__ Op<NT> load_rows(const double* M, int rows, int cols, int t) {
    Op<NT> o;
#pragma unroll
    for (int s = 0; s < NT; ++s) o.f[s] = load_tile_t(M + (int64_t)16 * t * cols + 16 * s, rows - 16 * t, cols - 16 * s, cols);
    return o;
}
template <int NT>
__device__ __forceinline__ f64x4 apply(const Op<NT>& o, const f64x4 (&all)[NT], f64x4 acc) {
#pragma unroll
    for (int s = 0; s < NT; ++s) acc = mm(o.f[s], all[s], acc);
    return acc;
}
template <int NT, typename T>
__device__ __forceinline__ void load_all(const T* x, int n, f64x4 (&all)[NT]) {
#pragma unroll
    for (int s = 0; s < NT; ++s) all[s] = load_vec(x + 16 * s, n - 16 * s);
}
template <typename T>
__device__ __forceinline__ void store_own(T* x, const f64x4& v, int n, int t) { store_col<4>(x + 16 * t, v, n - 16 * t); }
template <typename T>
__device__ __forceinline__ f64x4 load_own(const T* x, int n, int t) { return load_vec(x + 16 * t, n - 16 * t); }

template <bool UP, int D, int NT>
__device__ __forceinline__ f64x4 scan_level(Rows<NT>& w, const f64x4& X, const double* M, int n) {
    f64x4 all[NT];
    w.share(X, all);
#pragma unroll
    for (int s = 0; s < NT; ++s) all[s] = shift<UP, D, 4>(all[s]);
    return apply(load_rows<NT>(M, n, n, w.t), all, X);
}
// inclusive scan over the columns (see steady.hip)
template <bool UP, int NT>
__device__ __forceinline__ f64x4 column_scan(Rows<NT>& w, f64x4 X, const double* mp, int n) {
    const int n2 = n * n;
    X = scan_level<UP, 1>(w, X, mp, n);
    X = scan_level<UP, 2>(w, X, mp + n2, n);
    X = scan_level<UP, 4>(w, X, mp + 2 * n2, n);
    return scan_level<UP, 8>(w, X, mp + 3 * n2, n);
}
template <bool UP, int NT>
__device__ __forceinline__ f64x4 column_spread(Rows<NT>& w, const f64x4& v, const double* mp, int n) {
    f64x4 X;
    const bool edge = lane_i() == (UP ? 0 : 15);
#pragma unroll
    for (int i = 0; i < 4; ++i) X[i] = edge ? v[i] : 0.0;
    return column_scan<UP>(w, X, mp, n);
}

struct ChainL {
    int64_t start, len, k0;
};
__device__ __forceinline__ ChainL chain_of(const Args& a, int nh, int64_t tile) {
    ChainL c;
    const int b = a.B > 1 ? seq_holding(a.blk_off, a.B, tile) : 0;
    const SeqR q = seq_of(a, b);
    c.start = q.start;
    c.len = q.end - q.start;
    c.k0 = nh + (((tile - a.blk_off[b]) * 16 + lane_i()) << a.pL);
    return c;
}

template <typename R, int NT, bool STORE>
__device__ __forceinline__ f64x4 run_filter(const Args& a, Rows<NT>& w, const Head& h, int run, f64x4 X, f64x4 (&rows)[kRun]) {
    const int n = a.nx, m = a.ny;
    const R* y = static_cast<const R*>(a.y) + h.start * m;
    R* mo = static_cast<R*>(a.m) + h.start * n;
#pragma unroll 1
    for (int j = 0; j < kRun; ++j) {
        const int k = run * kRun + j;
        const Op<NT> phi = load_rows<NT>(a.tPhi + (int64_t)k * n * n, n, n, w.t);
        const Op<NT> kk = load_rows<NT>(a.tK + (int64_t)k * n * m, n, m, w.t);
        f64x4 all[NT];
        load_all<NT>(y + (int64_t)(k < h.len ? k : 0) * m, k < h.len ? m : 0, all);
        const f64x4 gain = apply(kk, all, load_own(a.tc + (int64_t)k * n, n, w.t));
        w.share(X, all);
        X = apply(phi, all, gain);
        if constexpr (STORE) {
#pragma unroll
            for (int i = 0; i < kRun; ++i)
                if (i == j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) rows[i][v] = double(R(X[v]));
            if (k < h.len) store_own(mo + (int64_t)k * n, X, n, w.t);
        }
    }
    return X;
}
template <typename R, int NT, bool STORE>
__device__ __forceinline__ f64x4 run_smoother(const Args& a, Rows<NT>& w, const Head& h, int run, f64x4 Z, const f64x4 (&mk)[kRun]) {
    const int n = a.nx, n2 = n * n;
    R* mo = static_cast<R*>(a.ms) + h.start * n;
    const Op<NT> F = load_rows<NT>(a.F, n, n, w.t);
    const f64x4 u = a.u ? load_own(a.u, n, w.t) : zero4();
#pragma unroll 1
    for (int j = kRun - 1; j >= 0; --j) {
        const int k = run * kRun - 1 + j;
        if (k < 0) break;
        f64x4 own = mk[0], all[NT];
#pragma unroll
        for (int i = 1; i < kRun; ++i)
            if (i == j) own = mk[i];
        const Op<NT> E = load_rows<NT>(a.tE + (int64_t)k * n2, n, n, w.t);
        w.share(own, all);
        const f64x4 p = apply(F, all, u);
        w.share(Z - p, all);
        const f64x4 Zn = apply(E, all, own);
#pragma unroll
        for (int v = 0; v < 4; ++v) Z[v] = k >= h.full ? 0.0 : (k == h.full - 1 ? own[v] : Zn[v]);
        if constexpr (STORE)
            if (k < h.len) store_own(mo + (int64_t)k * n, Z, n, w.t);
    }
    return Z;
}

// the filtered means that a run of a head smooths
template <typename R, int NT>
__device__ __forceinline__ void head_means(const Args& a, const Rows<NT>& w, const Head& h, int run, f64x4 (&mk)[kRun]) {
    const R* mi = static_cast<const R*>(a.m) + h.start * a.nx;
#pragma unroll
    for (int j = 0; j < kRun; ++j) {
        const int k = run * kRun - 1 + j;
        mk[j] = k >= 0 && k < h.len ? load_own(mi + (int64_t)k * a.nx, a.nx, w.t) : zero4();
    }
}

struct GridL {
    int64_t heads, tiles;
};
__device__ __forceinline__ bool head_of_block(const Args& a, int nh, int64_t id, int& group, int& run) {
    const int nrun = nh / kRun;
    group = (int)(id / nrun);
    run = (int)(id % nrun);
    return group * 16 < a.B;
}

// chains and head runs of the filter from zero; P
template <typename R, int NT>
__global__ __launch_bounds__(64 * NT) void k_stl_filter_reduce(Args a, GridL g) {
    __shared__ f64x4 buf[2][NT][64];
    extern __shared__ __align__(16) double dyn[];
    const int nh = a.ctl[0];
    if (nh == 0) return;
    const int n = a.nx, m = a.ny;
    Rows<NT> w(buf);
    int64_t blk = blockIdx.x;
    if (blk < g.heads) {
        int group, run;
        if (!head_of_block(a, nh, blk, group, run)) return;
        const Head h = head_of(a, nh, group);
        f64x4 rows[kRun];
        const f64x4 X = run_filter<R, NT, false>(a, w, h, run, zero4(), rows);
        if (h.full > 0) store_own(run_vec(a, a.runB, h.b, run), X, n, w.t);
        return;
    }
    blk -= g.heads;
    if (blk >= g.tiles) {
        write_rows<R, false>(a, nh, blk - g.tiles, gridDim.x - g.heads - g.tiles, reinterpret_cast<R*>(dyn));
        return;
    }
    if (blk >= a.blk_off[a.B]) return;
    const ChainL c = chain_of(a, nh, blk);
    const R* y = static_cast<const R*>(a.y) + c.start * m;
    const Op<NT> Phi = load_rows<NT>(a.star + star_Phi(n, m), n, n, w.t), K = load_rows<NT>(a.star + star_K(n, m), n, m, w.t);
    const f64x4 cc = load_own(a.star + star_c(n, m), n, w.t);
    const int64_t last = c.len - 1;
    const int L = 1 << a.pL;
    f64x4 X = zero4(), yn[NT], all[NT];
    auto at = [&](int64_t k, f64x4 (&v)[NT]) { load_all<NT>(y + (k < last ? k : last) * m, m, v); };
    at(c.k0, yn);
    for (int i = 0; i < L; ++i) {
        const f64x4 gain = apply(K, yn, cc);
        at(c.k0 + i + 1, yn);
        w.share(X, all);
        X = apply(Phi, all, gain);
    }
    X = column_scan<true>(w, X, a.mpF, n);
    store_own(a.pre + (blk * 16 + lane_i()) * n, shift<true, 1, 4>(X), n, w.t);
    if (lane_i() == 15) store_own(a.agg + blk * n, X, n, w.t);
}

// One sequence: what enters each of its tiles and each run of its head
template <typename R, int NT, bool REV>
__global__ __launch_bounds__(64 * NT) void k_stl_top(Args a) {
    __shared__ f64x4 buf[2][NT][64];
    const int nh = a.ctl[0];
    if (nh == 0) return;
    const int n = a.nx, n2 = n * n, b = blockIdx.x, li = lane_i();
    Rows<NT> w(buf);
    const SeqR sq = seq_of(a, b);
    const int64_t len = sq.end - sq.start;
    const int64_t t0 = a.blk_off[b], nt = a.blk_off[b + 1] - t0;
    const int nrun = nh / kRun;
    const double* mp = (REV ? a.mpE : a.mpF) + (int64_t)4 * n2;
    const double* runM = REV ? a.runE : a.runPhi;
    auto tile_at = [&](int64_t i) { return REV ? t0 + nt - 1 - i : t0 + i; };
    auto run_at = [&](int i) { return REV ? nrun - 1 - i : i; };
    f64x4 all[NT];
    auto head = [&](f64x4 X) {
        Op<NT> next = load_rows<NT>(runM + (int64_t)run_at(0) * n2, n, n, w.t);
        f64x4 Vn = load_own(run_vec(a, a.runB, b, run_at(0)), n, w.t);
        for (int i = 0; i < nrun; ++i) {
            const Op<NT> op = next;
            const f64x4 V = Vn;
            const int in = run_at(i + 1 < nrun ? i + 1 : i);
            next = load_rows<NT>(runM + (int64_t)in * n2, n, n, w.t);
            Vn = load_own(run_vec(a, a.runB, b, in), n, w.t);
            if (li == 0) store_own(run_vec(a, a.runX, b, run_at(i)), X, n, w.t);
            w.share(X, all);
            X = apply(op, all, V);
        }
        return X;
    };
    f64x4 X = zero4();
    if constexpr (!REV) X = head(load_own(a.m0, n, w.t));
    const Op<NT> M = load_rows<NT>(mp + (int64_t)4 * n2, n, n, w.t);
    for (int64_t i0 = 0; i0 < nt; i0 += 16) {       // 16 tiles at a time
        const int64_t i = i0 + li;
        const f64x4 A = column_scan<true>(w, i < nt ? load_own(a.agg + tile_at(i) * n, n, w.t) : zero4(), mp, n);
        const f64x4 in = shift<true, 1, 4>(A) + column_spread<true>(w, X, mp, n);
        if (i < nt) store_own(a.car + tile_at(i) * n, in, n, w.t);
        f64x4 sum;
#pragma unroll
        for (int v = 0; v < 4; ++v) sum[v] = col_bcast(A[v], 15);
        w.share(X, all);
        X = apply(M, all, sum);
    }
    if constexpr (REV) {
        __syncthreads();
        X = zero4();
        if (len >= nh) {
            const f64x4 mk = load_own(static_cast<const R*>(a.m) + (sq.start + nh - 1) * n, n, w.t);
            X = mk;
            if (len > nh) {
                load_all<NT>(a.car + t0 * n, n, all);
                const f64x4 Z = apply(load_rows<NT>(mp, n, n, w.t), all, load_own(a.agg + t0 * n, n, w.t));
                w.share(mk, all);
                const f64x4 p = apply(load_rows<NT>(a.F, n, n, w.t), all, a.u ? load_own(a.u, n, w.t) : zero4());
                w.share(Z - p, all);
                X = apply(load_rows<NT>(a.star + star_E(n, a.ny), n, n, w.t), all, mk);
            }
        }
        head(X);
    }
}

// filtered means; the chains and head runs of the smoother from zero, backwards
template <typename R, int NT>
__global__ __launch_bounds__(64 * NT) void k_stl_filter_down(Args a, GridL g) {
    __shared__ f64x4 buf[2][NT][64];
    const int nh = a.ctl[0];
    if (nh == 0) return;
    const int n = a.nx, m = a.ny;
    Rows<NT> w(buf);
    int64_t blk = blockIdx.x;
    if (blk < g.heads) {
        int group, run;
        if (!head_of_block(a, nh, blk, group, run)) return;
        const Head h = head_of(a, nh, group);
        f64x4 rows[kRun], mk[kRun];
        if (a.given) {
            head_means<R, NT>(a, w, h, run, mk);
        } else {
            const f64x4 X0 = load_own(run_vec(a, a.runX, h.b, run), n, w.t);
            run_filter<R, NT, true>(a, w, h, run, X0, rows);
            if (!a.smooth) return;
#pragma unroll
            for (int v = 0; v < 4; ++v) mk[0][v] = double(R(X0[v]));
#pragma unroll
            for (int j = 1; j < kRun; ++j) mk[j] = rows[j - 1];
        }
        const f64x4 Z = run_smoother<R, NT, false>(a, w, h, run, zero4(), mk);
        if (h.full > 0) store_own(run_vec(a, a.runB, h.b, run), Z, n, w.t);
        return;
    }
    blk -= g.heads;
    if (blk >= a.blk_off[a.B]) return;
    const ChainL c = chain_of(a, nh, blk);
    const R* y = static_cast<const R*>(a.y) + c.start * m;
    R* mo = static_cast<R*>(a.m) + c.start * n;
    const int64_t last = c.len - 1;
    const int L = 1 << a.pL;
    double* pre = a.pre + (blk * 16 + lane_i()) * n;
    f64x4 all[NT];
    if (!a.given) {
        const Op<NT> Phi = load_rows<NT>(a.star + star_Phi(n, m), n, n, w.t);
        const Op<NT> K = load_rows<NT>(a.star + star_K(n, m), n, m, w.t);
        const f64x4 cc = load_own(a.star + star_c(n, m), n, w.t);
        f64x4 yn[NT];
        auto at = [&](int64_t k, f64x4 (&v)[NT]) { load_all<NT>(y + (k < last ? k : last) * m, m, v); };
        at(c.k0, yn);
        f64x4 X = load_own(pre, n, w.t) + column_spread<true>(w, load_own(a.car + blk * n, n, w.t), a.mpF, n);
        for (int i = 0; i < L; ++i) {
            const f64x4 gain = apply(K, yn, cc);
            at(c.k0 + i + 1, yn);
            w.share(X, all);
            X = apply(Phi, all, gain);
            if (c.k0 + i <= last) store_own(mo + (c.k0 + i) * n, X, n, w.t);
        }
    }
    if (!a.smooth) return;
    __threadfence_block();
    __syncthreads();               // every wave's rows of the means are read below
    const Op<NT> F = load_rows<NT>(a.F, n, n, w.t), E = load_rows<NT>(a.star + star_E(n, m), n, n, w.t);
    const f64x4 u = a.u ? load_own(a.u, n, w.t) : zero4();
    f64x4 Z = zero4(), mn[NT];
    auto at = [&](int64_t k, f64x4 (&v)[NT]) { load_all<NT>(mo + (k < last ? k : last) * n, n, v); };
    at(c.k0 + L - 1, mn);
    for (int i = L - 1; i >= 0; --i) {
        const int64_t k = c.k0 + i;
        const f64x4 p = apply(F, mn, u);
        f64x4 mk = mn[0];
#pragma unroll
        for (int s = 1; s < NT; ++s)
            if (s == w.t) mk = mn[s];
        at(c.k0 + (i > 0 ? i - 1 : 0), mn);
        w.share(Z - p, all);
        const f64x4 Zn = apply(E, all, mk);
#pragma unroll
        for (int v = 0; v < 4; ++v) Z[v] = k > last ? 0.0 : (k == last ? mk[v] : Zn[v]);
    }
    Z = column_scan<false>(w, Z, a.mpE, n);
    store_own(pre, shift<false, 1, 4>(Z), n, w.t);
    if (lane_i() == 0) store_own(a.agg + blk * n, Z, n, w.t);
}

// smoothed means; Ps
template <typename R, int NT>
__global__ __launch_bounds__(64 * NT) void k_stl_smoother_down(Args a, GridL g) {
    __shared__ f64x4 buf[2][NT][64];
    extern __shared__ __align__(16) double dyn[];
    const int nh = a.ctl[0];
    if (nh == 0) return;
    const int n = a.nx, m = a.ny;
    Rows<NT> w(buf);
    int64_t blk = blockIdx.x;
    if (blk < g.heads) {
        int group, run;
        if (!head_of_block(a, nh, blk, group, run)) return;
        const Head h = head_of(a, nh, group);
        f64x4 mk[kRun];
        head_means<R, NT>(a, w, h, run, mk);
        const f64x4 Z = load_own(run_vec(a, a.runX, h.b, run), n, w.t);
        if ((run + 1) * kRun == nh && h.len == nh)
            store_own(static_cast<R*>(a.ms) + (h.start + nh - 1) * n, Z, n, w.t);
        run_smoother<R, NT, true>(a, w, h, run, Z, mk);
        return;
    }
    blk -= g.heads;
    if (blk >= g.tiles) {
        write_rows<R, true>(a, nh, blk - g.tiles, gridDim.x - g.heads - g.tiles, reinterpret_cast<R*>(dyn));
        return;
    }
    if (blk >= a.blk_off[a.B]) return;
    const ChainL c = chain_of(a, nh, blk);
    const R* mi = static_cast<const R*>(a.m) + c.start * n;
    R* mo = static_cast<R*>(a.ms) + c.start * n;
    const int64_t last = c.len - 1;
    const int L = 1 << a.pL;
    const Op<NT> F = load_rows<NT>(a.F, n, n, w.t), E = load_rows<NT>(a.star + star_E(n, m), n, n, w.t);
    const f64x4 u = a.u ? load_own(a.u, n, w.t) : zero4();
    f64x4 all[NT], mn[NT];
    auto at = [&](int64_t k, f64x4 (&v)[NT]) { load_all<NT>(mi + (k < last ? k : last) * n, n, v); };
    at(c.k0 + L - 1, mn);
    f64x4 Z = load_own(a.pre + (blk * 16 + lane_i()) * n, n, w.t) +
              column_spread<false>(w, load_own(a.car + blk * n, n, w.t), a.mpE, n);
    for (int i = L - 1; i >= 0; --i) {
        const int64_t k = c.k0 + i;
        const f64x4 p = apply(F, mn, u);
        f64x4 mk = mn[0];
#pragma unroll
        for (int s = 1; s < NT; ++s)
            if (s == w.t) mk = mn[s];
        at(c.k0 + (i > 0 ? i - 1 : 0), mn);
        w.share(Z - p, all);
        const f64x4 Zn = apply(E, all, mk);
        if (k <= last) {
            Z = k == last ? mk : Zn;
            store_own(mo + k * n, Z, n, w.t);
        }
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
template <typename K>
hipError_t allow(K kernel, size_t lds) {
    if (lds <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

template <typename R, int NT>
hipError_t run(const Args& a, hipStream_t s) {
    const int writers = 1024, runs = a.N / kRun;
    const size_t eng = sizeof(double) * Eng<NT>::kLds, row = sizeof(R) * a.nx * a.nx;
    const dim3 wide(64 * NT * NT), block(64 * NT);
    hipError_t e;
    if ((e = allow(k_stl_double<NT>, eng)) != hipSuccess || (e = allow(k_stl_tables<NT>, eng)) != hipSuccess ||
        (e = allow(k_stl_head_scan<NT>, eng)) != hipSuccess || (e = allow(k_stl_head_fill<NT>, eng)) != hipSuccess ||
        (e = allow(k_stl_short_head<R, NT>, eng)) != hipSuccess)
        return e;
    if (a.given) {
        prof_begin("k_stl_probe", s);
        hipLaunchKernelGGL((k_stl_probe<R>), dim3(1), dim3(256), 0, s, a);
        prof_end(s);
    }
    prof_begin("k_stl_double", s);
    hipLaunchKernelGGL((k_stl_double<NT>), dim3(1), wide, eng, s, a);
    prof_end(s);
    prof_begin("k_stl_tables", s);
    hipLaunchKernelGGL((k_stl_tables<NT>), dim3(2 + (a.smooth ? 2 : 1) * runs), wide, eng, s, a);
    prof_end(s);
    if (a.smooth) {
        const double *sE = a.runE, *sL = a.runL;
        int at = 0;
        for (int d = 1; d < runs; d <<= 1) {
            prof_begin("k_stl_head_scan", s);
            hipLaunchKernelGGL((k_stl_head_scan<NT>), dim3(runs), wide, eng, s, a, sE, sL, a.scanE[at], a.scanL[at], d);
            prof_end(s);
            sE = a.scanE[at];
            sL = a.scanL[at];
            at ^= 1;
        }
        prof_begin("k_stl_head_fill", s);
        hipLaunchKernelGGL((k_stl_head_fill<NT>), dim3(runs), wide, eng, s, a, sE, sL);
        prof_end(s);
        prof_begin("k_stl_short_head", s);
        if (a.B > 1) hipLaunchKernelGGL((k_stl_short_head<R, NT>), dim3(a.B, runs), wide, eng, s, a);
        prof_end(s);
    }
    const GridL g{(int64_t)((a.B + 15) / 16) * runs, a.max_blocks};
    const dim3 chains((unsigned)(g.heads + g.tiles)), with_rows((unsigned)(g.heads + g.tiles + writers));
    if (a.given) {
        prof_begin("k_stl_check", s);
        hipLaunchKernelGGL((k_stl_check<R>), dim3(writers), dim3(256), row, s, a);
        prof_end(s);
    } else {
        prof_begin("k_stl_filter_reduce", s);
        hipLaunchKernelGGL((k_stl_filter_reduce<R, NT>), with_rows, block, row, s, a, g);
        prof_end(s);
        prof_begin("k_stl_filter_top", s);
        hipLaunchKernelGGL((k_stl_top<R, NT, false>), dim3(a.B), block, 0, s, a);
        prof_end(s);
    }
    prof_begin("k_stl_filter_down", s);
    hipLaunchKernelGGL((k_stl_filter_down<R, NT>), chains, block, 0, s, a, g);
    prof_end(s);
    if (a.smooth) {
        prof_begin("k_stl_smoother_top", s);
        hipLaunchKernelGGL((k_stl_top<R, NT, true>), dim3(a.B), block, 0, s, a);
        prof_end(s);
        prof_begin("k_stl_smoother_down", s);
        hipLaunchKernelGGL((k_stl_smoother_down<R, NT>), with_rows, block, row, s, a, g);
        prof_end(s);
    }
    return hipGetLastError();
}

template <typename R>
hipError_t run_nt(const Args& a, hipStream_t s) {
    switch ((a.nx + 15) / 16) {
        case 2: return run<R, 2>(a, s);
        case 3: return run<R, 3>(a, s);
        default: return run<R, 4>(a, s);
    }
}

}  // namespace

hipError_t launch_large(const Args& a, bool mixed, hipStream_t s) { return mixed ? run_nt<float>(a, s) : run_nt<double>(a, s); }

}  // namespace steady
}  // namespace pks
