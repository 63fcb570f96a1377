// Whole solves of 2D grids that fit one CU: one workgroup per load case keeps the
// search direction, the spectrum, the residual, u and, for finite
// strain, the displacement in LDS and runs the CG (or Newton with its CG) to
// the end in one launch.
//
// On a small grid an iteration of the general path is six to eight dependent
// launches, each as long as one workgroup's latency (about 5 us), however
// little it computes; here it is some twenty barriers.  The arithmetic is that
// of the general path: plan precision for the stencil of the small-strain
// solve, the transforms and M^-1, FP64 for every sum and for the finite-strain
// stress.
// Bound: LDS latency and barriers.
// Measured against the general path, random materials of contrast 10: solve of
// 3 load cases to 1e-10 in FP64, 8^2 0.90 -> 0.23 ms, 17^2 1.52 -> 0.48,
// 33^2 1.65 -> 0.99, 48^2 1.49 -> 0.89; to 1e-5 in FP32, 64^2 0.83 -> 0.62;
// finite strain of one load case to 1e-8 in FP64, 17^2 3.34 -> 1.22,
// 40^2 4.36 -> 2.07.  Over 152 solves of 1 to 64 load cases and 64 finite-strain
// solves, squares to 64^2 and strips to 2 x 1021, it was 1.3 to 5.4 times as
// fast wherever it fits, so the rule is what fits: the LDS, the points a thread
// may hold in a pass and the matrix-core tiles of the prime passes (odd rows
// take twice the room of even ones).  Largest squares, even and odd: FP64 48^2
// and 33^2, FP32 64^2 and 47^2; finite strain FP64 40^2 and 33^2, FP32 50^2 and
// 47^2.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "fft_butterflies.hpp"
#include "nodal_stencil.hpp"

namespace feh {
namespace {

constexpr int DIM = 2, NT = 512, NW = NT / 64;
constexpr size_t kLdsUse = 150 * 1024;
extern __shared__ double small_lds[];

// Complex points of a transform that a thread may hold.
template <typename T>
constexpr int kPoints = sizeof(T) == 4 ? 10 : 5;
constexpr int kTiles = 4;  // matrix-core tiles of a prime pass a wavefront may hold

// One axis of the spectrum in LDS: batch b = (hi, lo) at hi * A + lo, element
// j of it at j * stride beyond.
struct Axis {
    AxisFFT fft;
    FastDiv nb, lo;     // batches; extent of lo
    int A, stride, tws;
};

template <typename T>
struct SmallArgs {
    Axis ax[2];
    const Cx<T> *tw[2];     // e^{-2 pi i j / n_a}
    const T *lam, *mu, *minv;
    const double *Ebar;     // small strain: Ebar; finite strain: the final Fbar, [L][D][D]
    void *u;                // small strain: [L][D][N] of the kernel's U
    double *uf;             // finite strain: [L][D][N]
    double *fbar;           // finite strain: the last load step's Fbar
    double *fin;            // finite strain: [L][5] newton, cg, status, rel_equilibrium, rel_increment
    LcState *st;
    int G;                  // load cases per material
    int n[3], N, rows, nlast, nc, nh, S, even, inner, nspec;
    FastDiv d_N, d_last, d_nh, d_inner, d_D, d_half;
    int table_lds, mat_lds;  // the table of inverses, the material kept in LDS
    T ih[3], vol;
    double ihd[3], w, invN, tol;
    int max_iter;
    int n_steps, max_newton;
    double newton_tol, equil_tol;
};

__device__ __forceinline__ int batch_base(const Axis &x, int b) {
    const int hi = (int)x.lo.div((uint32_t)b);
    return hi * x.A + (b - hi * (int)x.lo.d);
}

template <typename T, int R>
__device__ __forceinline__ void small_pass(Cx<T> *W, const Axis &x, const PassInfo &ps, const Cx<T> *tw, bool inv) {
    constexpr int K = (kPoints<T> + R - 1) / R;
    const int nb = (int)x.nb.d, n = x.fft.n, m = (int)ps.m.d, total = nb * (n / R);
    Cx<T> y[K][R];
    int at[K];
    #pragma unroll
    for (int k = 0; k < K; ++k) {
        const int t = (int)threadIdx.x + k * NT;
        at[k] = -1;
        if (t < total) {
            const int w = (int)x.nb.div((uint32_t)t), b = t - w * nb;
            const int p = (int)ps.m.div((uint32_t)w), q = w - p * m;
            const int base = batch_base(x, b);
            Cx<T> v[R];
            #pragma unroll
            for (int c = 0; c < R; ++c) v[c] = W[base + (q + m * R * p + c * m) * x.stride];
            if (p != 0) {
                #pragma unroll
                for (int c = 1; c < R; ++c) v[c] = cmul(v[c], twid(tw, x.tws, c * p * m, inv));
            }
            Dft<T, R>::run(v, inv, tw, x.tws, n);
            #pragma unroll
            for (int d = 0; d < R; ++d) y[k][d] = v[d];
            at[k] = base + (q + m * p) * x.stride;
        }
    }
    __syncthreads();
    #pragma unroll
    for (int k = 0; k < K; ++k) {
        if (at[k] >= 0) {
            #pragma unroll
            for (int d = 0; d < R; ++d) W[at[k] + d * m * ps.Lstar * x.stride] = y[k][d];
        }
    }
    __syncthreads();
}

// Odd prime radix as two real products on the matrix cores; see prime_pass of
// the general passes for the formulas.
template <typename T>
__device__ __forceinline__ void small_prime(Cx<T> *W, const Axis &x, const PassInfo &ps, const Cx<T> *tw, bool inv) {
    using M = Mfma<T>;
    const int nb = (int)x.nb.d, n = x.fft.n, R = ps.R, m = (int)ps.m.d, Ls = ps.Lstar, H = (R - 1) / 2;
    const int nR = n / R, bf = nb * nR, cs = m * x.stride, os = m * Ls * x.stride, tx = threadIdx.x;
    auto place = [&](int w, int &p, int &q) {
        const int r = (int)x.nb.div((uint32_t)w);
        p = (int)ps.m.div((uint32_t)r);
        q = r - p * m;
        return batch_base(x, w - r * nb);
    };
    for (int i = tx; i < bf * H; i += NT) {
        const int c = 1 + i / bf, w = i - (c - 1) * bf;
        int p, q;
        const int base = place(w, p, q);
        Cx<T> *x0 = W + base + (q + m * R * p) * x.stride;
        Cx<T> a = x0[c * cs], b = x0[(R - c) * cs];
        if (p != 0) {
            a = cmul(a, twid(tw, x.tws, c * p * m, inv));
            b = cmul(b, twid(tw, x.tws, (R - c) * p * m, inv));
        }
        x0[c * cs] = cadd(a, b);
        x0[(R - c) * cs] = csub(a, b);
    }
    __syncthreads();
    const int lane = tx & 63, wv = tx >> 6, li = lane & 15, lg = lane >> 4;
    const int KT = (H + 1 + 15) / 16, CT = (2 * bf + 15) / 16;
    typename M::Acc A[kTiles], B[kTiles];
    T *re = reinterpret_cast<T *>(W);
    #pragma unroll
    for (int i = 0; i < kTiles; ++i) {
        const int t = wv + NW * i;
        if (t < KT * CT) {  // the same for the whole wavefront
            const int ct = t / KT, kt = t - ct * KT;
            const int col = ct * 16 + li;
            const bool on = (col >> 1) < bf;
            int p, q;
            const int base = place(on ? col >> 1 : 0, p, q);
            const T *x0 = re + 2 * (base + (q + m * R * p) * x.stride) + (col & 1);
            const int k = min(kt * 16 + li, H);
            const T first = on ? x0[0] : T(0);
            typename M::Acc a = {first, first, first, first}, b = {T(0), T(0), T(0), T(0)};
            int c = 1 + lg, e = (c * k) % R;
            const int step = (4 * k) % R;
            for (int c0 = 1; c0 <= H; c0 += 4) {
                const Cx<T> wt = tw[e * nR * x.tws];  // cos, -sin
                const bool in = on && c <= H;
                const int cc = in ? c : 1;
                const T sv = x0[2 * cc * cs], dv = x0[2 * (R - cc) * cs];
                a = M::run(wt.x, in ? sv : T(0), a);
                b = M::run(-wt.y, in ? dv : T(0), b);
                c += 4;
                e += step;
                if (e >= R) e -= R;
            }
            A[i] = a;
            B[i] = b;
        }
    }
    __syncthreads();
    #pragma unroll
    for (int i = 0; i < kTiles; ++i) {
        const int t = wv + NW * i;
        if (t < KT * CT) {
            const int ct = t / KT, kt = t - ct * KT;
            const int col = ct * 16 + li;
            const bool on = (col >> 1) < bf;
            int p, q;
            const int base = place(on ? col >> 1 : 0, p, q);
            T *y0 = re + 2 * (base + (q + m * p) * x.stride) + (col & 1);
            #pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k = kt * 16 + M::row(lane, r);
                const T bx = __shfl_xor(B[i][r], 1);
                const T ib = ((col & 1) != 0) == inv ? bx : -bx;
                if (on && k <= H) {
                    y0[2 * k * os] = A[i][r] + ib;
                    if (k > 0) y0[2 * (R - k) * os] = A[i][r] - ib;
                }
            }
        }
    }
    __syncthreads();
}

template <typename T>
__device__ __forceinline__ void small_fft(Cx<T> *W, const Axis &x, const int *pass, const Cx<T> *tw, bool inv) {
    for (int s = 0; s < x.fft.npass; ++s) {
        const int *o = pass + 5 * s;
        auto field = [&](int i) { return __builtin_amdgcn_readfirstlane(o[i]); };  // the same in every lane
        PassInfo ps;
        ps.R = field(0);
        ps.Lstar = field(1);
        ps.m.d = (uint32_t)field(2);
        ps.m.mul = (uint32_t)field(3);
        ps.m.sh = (uint32_t)field(4);
        switch (ps.R) {
        case 2: small_pass<T, 2>(W, x, ps, tw, inv); break;
        case 3: small_pass<T, 3>(W, x, ps, tw, inv); break;
        case 4: small_pass<T, 4>(W, x, ps, tw, inv); break;
        case 5: small_pass<T, 5>(W, x, ps, tw, inv); break;
        case 8: small_pass<T, 8>(W, x, ps, tw, inv); break;
        default: small_prime<T>(W, x, ps, tw, inv); break;  // 7, 11, 13 and larger primes
        }
    }
}

// Forward transform of the real field in W (rows packed two values to a point
// when the last axis is even, value and zero when it is odd).
template <typename T>
__device__ __forceinline__ void forward(const SmallArgs<T> &a, Cx<T> *W, const Cx<T> *const (&tw)[2], int *const (&pass)[2]) {
    small_fft<T>(W, a.ax[DIM - 1], pass[DIM - 1], tw[DIM - 1], false);
    if (a.even) {
        // points k and nc - k from one another
        const int half = a.nc / 2 + 1, total = a.rows * DIM * half;
        for (int i = threadIdx.x; i < total; i += NT) {
            const int rc = (int)a.d_half.div((uint32_t)i), k = i - rc * half;
            const int row = (int)a.d_D.div((uint32_t)rc);
            Cx<T> *x = W + row * a.S * DIM + (rc - row * DIM);
            const int km = a.nc - k;
            const Cx<T> Zk = x[k * DIM], Zm = k == 0 ? Zk : x[km * DIM];
            auto out = [&](Cx<T> z, Cx<T> zm, int kx) {
                zm = cconj(zm);
                const Cx<T> s = {T(0.5) * (z.x + zm.x), T(0.5) * (z.y + zm.y)};
                const Cx<T> d = csub(z, zm);
                return cadd(s, cmul(tw[DIM - 1][kx], Cx<T>{T(0.5) * d.y, -T(0.5) * d.x}));
            };
            x[k * DIM] = out(Zk, Zm, k);
            if (km != k) x[km * DIM] = out(Zm, Zk, km);
        }
        __syncthreads();
    }
    small_fft<T>(W, a.ax[0], pass[0], tw[0], false);
}

// The inverse (times N); imaginary parts of the real modes are dropped.
template <typename T>
__device__ __forceinline__ void inverse(const SmallArgs<T> &a, Cx<T> *W, const Cx<T> *const (&tw)[2], int *const (&pass)[2]) {
    small_fft<T>(W, a.ax[0], pass[0], tw[0], true);
    const int half = a.even ? a.nc / 2 + 1 : a.nh, total = a.rows * DIM * half;
    for (int i = threadIdx.x; i < total; i += NT) {
        const int rc = (int)a.d_half.div((uint32_t)i), k = i - rc * half;
        const int row = (int)a.d_D.div((uint32_t)rc);
        Cx<T> *x = W + row * a.S * DIM + (rc - row * DIM);
        if (a.even) {
            const int km = a.nc - k;
            Cx<T> Xk = x[k * DIM], Xm = x[km * DIM];
            if (k == 0) Xk.y = Xm.y = T(0);
            auto out = [&](Cx<T> z, Cx<T> zm, int kx) {
                zm = cconj(zm);
                return cadd(cadd(z, zm), mul_pi(cmulc(csub(z, zm), tw[DIM - 1][kx])));
            };
            x[k * DIM] = out(Xk, Xm, k);
            if (k != 0 && km != k) x[km * DIM] = out(Xm, Xk, km);
        } else if (k == 0) {
            x[0].y = T(0);
        } else {
            x[(a.nlast - k) * DIM] = cconj(x[k * DIM]);
        }
    }
    __syncthreads();
    small_fft<T>(W, a.ax[DIM - 1], pass[DIM - 1], tw[DIM - 1], true);
}

// Place in W (in reals) of component c of the field value i of its row.
template <typename T>
__device__ __forceinline__ int real_at(const SmallArgs<T> &a, int row, int i, int c) {
    return a.even ? 2 * ((row * a.S + (i >> 1)) * DIM + c) + (i & 1) : 2 * ((row * a.S + i) * DIM + c);
}

// Sum over the workgroup, in every thread (fixed order).  One barrier: calls
// take the two halves of `red` in turn (`turn` flips), so that a wavefront
// still summing one half is never overtaken by the next call's writes.
__device__ __forceinline__ double all_sum(double v, double *red, int &turn) {
    #pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    double *r = red + turn * NW;
    turn ^= 1;
    if ((threadIdx.x & 63) == 0) r[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = r[0];
    #pragma unroll
    for (int i = 1; i < NW; ++i) s += r[i];
    return s;
}

// Wavevector slot s = (i0, inner index): its place in W and weight in the
// half-spectrum Parseval sum.
template <typename T>
__device__ __forceinline__ int slot_at(const SmallArgs<T> &a, int s, double &weight) {
    const int row = (int)a.d_nh.div((uint32_t)s), kx = s - row * a.nh;  // row = (i0, i1)
    weight = kx == 0 || (a.even && kx == a.nh - 1) ? 1.0 : 2.0;
    return (row * a.S + kx) * DIM;
}

// z = M^-1 r at a slot; c-th entry of the inverse at m[c * stride].
template <typename T>
__device__ __forceinline__ double slot_solve(const T *m, int stride, const Cx<T> (&r)[DIM], Cx<T> (&z)[DIM]) {
    const Cx<T> o01 = {m[2 * stride], m[3 * stride]};
    z[0] = cadd(cscale(r[0], m[0]), cmul(o01, r[1]));
    z[1] = cadd(cmulc(r[0], o01), cscale(r[1], m[stride]));
    double dot = 0.0;
    #pragma unroll
    for (int c = 0; c < DIM; ++c) dot += double(r[c].x) * double(z[c].x) + double(r[c].y) * double(z[c].y);
    return dot;
}

// Values of the stencil's nodes around node (row, i) from an LDS field [D][N].
template <typename V>
__device__ __forceinline__ void lds_nodes(const Stencil &s, const V *f, int N, const Place<DIM> &pl, V (&u)[32][DIM]) {
    #pragma unroll
    for (int i = 0; i < 32; ++i) {
        if (i >= s.nn) break;
        const unsigned o = pl.at(s.node[i]);
        #pragma unroll
        for (int c = 0; c < DIM; ++c) u[i][c] = f[c * N + (int)o];
    }
}

// Small strain: column c of C : (Ebar + sym B p) at a point, in the plan
// precision; lam, mu carry the point's volume.
template <typename T, bool EB>
__device__ __forceinline__ void hooke_column(const Stencil &s, int slot, int c, const T (&p)[32][DIM], const T (&ih)[3], T lam,
                                             T mu, const T (&Eb)[DIM][DIM], T (&col)[DIM]) {
    auto g = [&](int i, int a) { return (p[s.plus[slot][a][0]][i] - p[s.minus[slot][a][0]][i]) * ih[a]; };
    T tr = T(0);
    #pragma unroll
    for (int j = 0; j < DIM; ++j) tr += g(j, j) + (EB ? Eb[j][j] : T(0));
    #pragma unroll
    for (int i = 0; i < DIM; ++i) {
        const T e2 = g(i, c) + g(c, i) + (EB ? T(2) * Eb[i][c] : T(0));  // 2 e_ic
        col[i] = i == c ? fma(lam, tr, mu * e2) : mu * e2;
    }
}

// LDS of a solve: P [D][N], W, R (the residual, [D][N]),
// X (u, or the increment; in U), [F: the displacement], reduction, material,
// twiddles, pass lists, table of inverses.  U: the type of X.
template <typename T, typename U, bool FINITE>
struct Lds {
    T *P, *R;
    Cx<T> *W;
    U *X;
    double *F, *red;
    const T *glam, *gmu;
    T *lam, *mu;
    bool in_lds;
    const Cx<T> *tw[2];
    int *pass[2];
    T *tab;
    __device__ __forceinline__ Lds(const SmallArgs<T> &a, long long material) {
        char *o = reinterpret_cast<char *>(small_lds);
        auto take = [&](int bytes) {
            char *at = o;
            o += (bytes + 15) & ~15;
            return at;
        };
        P = reinterpret_cast<T *>(take(DIM * a.N * (int)sizeof(T)));
        W = reinterpret_cast<Cx<T> *>(take(a.rows * a.S * DIM * (int)sizeof(Cx<T>)));
        R = reinterpret_cast<T *>(take(a.nspec * DIM * (int)sizeof(Cx<T>)));  // at least the N a component
        X = reinterpret_cast<U *>(take(DIM * a.N * (int)sizeof(U)));
        F = reinterpret_cast<double *>(take(FINITE ? DIM * a.N * 8 : 0));
        red = reinterpret_cast<double *>(take(2 * NW * 8));
        glam = a.lam + material;
        gmu = a.mu + material;
        in_lds = a.mat_lds != 0;
        lam = reinterpret_cast<T *>(take(in_lds ? a.N * (int)sizeof(T) : 0));
        mu = reinterpret_cast<T *>(take(in_lds ? a.N * (int)sizeof(T) : 0));
        if (in_lds)
            for (int i = threadIdx.x; i < a.N; i += NT) {
                lam[i] = glam[i];
                mu[i] = gmu[i];
            }
        #pragma unroll
        for (int x = 0; x < DIM; ++x) {
            Cx<T> *t = reinterpret_cast<Cx<T> *>(take(a.n[x] * (int)sizeof(Cx<T>)));
            for (int i = threadIdx.x; i < a.n[x]; i += NT) t[i] = a.tw[x][i];
            tw[x] = t;
            // by constant index: an index known only at run time would put the
            // kernel's arguments in scratch memory
            pass[x] = reinterpret_cast<int *>(take(5 * kMaxRadixCount * 4));
            if (threadIdx.x == 0) {
                #pragma unroll
                for (int i = 0; i < kMaxRadixCount; ++i) {
                    const PassInfo &ps = a.ax[x].fft.pass[i];
                    int *o = pass[x] + 5 * i;
                    o[0] = ps.R;
                    o[1] = ps.Lstar;
                    o[2] = (int)ps.m.d;
                    o[3] = (int)ps.m.mul;
                    o[4] = (int)ps.m.sh;
                }
            }
        }
        constexpr int NC = 4;
        tab = reinterpret_cast<T *>(take(a.table_lds ? NC * a.nspec * (int)sizeof(T) : 0));
        if (a.table_lds) {
            // plain table: entry c of pencil inn, index i0 at (inn NC + c) n0 + i0
            for (int s = threadIdx.x; s < a.nspec; s += NT) {
                const int i0 = (int)a.d_inner.div((uint32_t)s), inn = s - i0 * a.inner;
                for (int c = 0; c < NC; ++c) tab[c * a.nspec + s] = a.minv[(inn * NC + c) * a.n[0] + i0];
            }
        }
        __syncthreads();
    }
};

template <typename M, typename T>
__device__ __forceinline__ void material_at(const M &m, unsigned v, T &lam, T &mu) {
    lam = m.in_lds ? m.lam[v] : m.glam[v];
    mu = m.in_lds ? m.mu[v] : m.gmu[v];
}

// r -= alpha q, q in W; r into W for the transform.  The residual is kept as a
// real field: its rounding is then a real force, which the CG can balance, and
// the transforms' own enters the preconditioner alone.  (Kept transformed,
// r^ -= alpha q^, FP32 solves on even grids gathered rounding of 1e-7 of the
// first residual that no step could take out again: long grids diverged where
// the general path converges, 900 x 2 at 1e-6.)
template <typename T, typename M>
__device__ __forceinline__ void advance(const SmallArgs<T> &a, const M &m, double alpha) {
    T *w = reinterpret_cast<T *>(m.W);
    for (int e = threadIdx.x; e < DIM * a.N; e += NT) {
        const int c = (int)a.d_N.div((uint32_t)e), v = e - c * a.N;
        const int row = (int)a.d_last.div((uint32_t)v), i = v - row * a.nlast;
        T &q = w[real_at<T>(a, row, i, c)];
        q = T(fma(-T(alpha), q, m.R[e]));
        m.R[e] = q;
    }
    __syncthreads();
}

// W = z^ = M^-1 r^ for the spectrum r^ in W; returns r.z.
template <typename T, typename M>
__device__ __forceinline__ double precondition(const SmallArgs<T> &a, const M &m, int &turn) {
    constexpr int NC = 4;
    double acc = 0.0;
    for (int s = threadIdx.x; s < a.nspec; s += NT) {
        double wt;
        Cx<T> *x = m.W + slot_at<T>(a, s, wt);
        Cx<T> r[DIM], z[DIM];
        #pragma unroll
        for (int c = 0; c < DIM; ++c) r[c] = x[c];
        double d;
        if (a.table_lds) {
            d = slot_solve<T>(m.tab + s, a.nspec, r, z);
        } else {
            const int i0 = (int)a.d_inner.div((uint32_t)s), inn = s - i0 * a.inner;
            d = slot_solve<T>(a.minv + (inn * NC) * a.n[0] + i0, a.n[0], r, z);
        }
        #pragma unroll
        for (int c = 0; c < DIM; ++c) x[c] = z[c];
        acc += wt * d;
    }
    return all_sum(acc, m.red, turn) * a.invN;  // its barrier also orders W for the inverse
}

// p = z / N + beta p from the real field in W.
template <typename T, typename M>
__device__ __forceinline__ void direction(const SmallArgs<T> &a, const M &m, T beta) {
    const T *w = reinterpret_cast<const T *>(m.W);
    const T sc = T(a.invN);
    for (int e = threadIdx.x; e < DIM * a.N; e += NT) {
        const int c = (int)a.d_N.div((uint32_t)e), v = e - c * a.N;
        const int row = (int)a.d_last.div((uint32_t)v), i = v - row * a.nlast;
        const T z = w[real_at<T>(a, row, i, c)] * sc;
        m.P[e] = beta == T(0) ? z : fma(beta, m.P[e], z);
    }
    __syncthreads();
}

// Zeros of the padding that the transforms read: the imaginary parts of an odd
// row's values (written with each value below), nothing on even rows.
template <typename T>
__device__ __forceinline__ void put_real(const SmallArgs<T> &a, T *w, int row, int i, int c, T v) {
    const int o = real_at<T>(a, row, i, c);
    w[o] = v;
    if (!a.even) w[o + 1] = T(0);
}

template <typename T, typename U>
__global__ __launch_bounds__(NT) void k_small_solve(SmallArgs<T> a) {
    static constexpr Stencil s = make_stencil<DIM, FEH_DERIV_FE>();
    const int l = blockIdx.x;
    const Lds<T, U, false> m(a, (long long)(l / a.G) * a.N);
    T *w = reinterpret_cast<T *>(m.W);
    int turn = 0;
    T Eb[DIM][DIM];
    #pragma unroll
    for (int i = 0; i < DIM; ++i)
        #pragma unroll
        for (int j = 0; j < DIM; ++j) Eb[i][j] = T(a.Ebar[(l * DIM + i) * DIM + j]);
    // W = q = w B^T C B p (returns this thread's part of p.q), or the load vector
    auto apply = [&](auto load) __attribute__((always_inline)) {
        constexpr bool LOAD = decltype(load)::value;
        double acc = 0.0;
        for (int v = threadIdx.x; v < a.N; v += NT) {
            const Place<DIM> pl(a.n, (unsigned)v, a.d_last.div((uint32_t)v));
            T p[32][DIM];
            if constexpr (LOAD) {
                #pragma unroll
                for (int i = 0; i < 32; ++i)
                    #pragma unroll
                    for (int c = 0; c < DIM; ++c) p[i][c] = T(0);
            } else {
                lds_nodes<T>(s, m.P, a.N, pl, p);
            }
            T q[DIM];
            #pragma unroll
            for (int i = 0; i < DIM; ++i) q[i] = T(0);
            auto column = [&](int slot, int c, T (&col)[DIM]) __attribute__((always_inline)) {
                const unsigned vo = pl.at(s.vox[slot]);
                T lam, mu;
                material_at(m, vo, lam, mu);
                hooke_column<T, LOAD>(s, slot, c, p, a.ih, lam * a.vol, mu * a.vol, Eb, col);
            };
            #pragma unroll
            for (int k = 0; k < s.nb; ++k) {
                T e[DIM], b[DIM];
                column(s.end[k], s.axis[k], e);
                column(s.start[k], s.axis[k], b);
                #pragma unroll
                for (int i = 0; i < DIM; ++i) q[i] = fma(e[i] - b[i], a.ih[s.axis[k]], q[i]);
            }
            const int row = (int)a.d_last.div((uint32_t)v), i0 = v - row * a.nlast;
            #pragma unroll
            for (int i = 0; i < DIM; ++i) {
                put_real<T>(a, w, row, i0, i, LOAD ? -q[i] : q[i]);
                if constexpr (LOAD) m.R[i * a.N + v] = -q[i];
                if constexpr (!LOAD) acc += double(p[0][i]) * double(q[i]);
            }
        }
        return acc;
    };
    for (int e = threadIdx.x; e < DIM * a.N; e += NT) m.X[e] = U(0);
    apply(std::true_type{});
    __syncthreads();
    forward<T>(a, m.W, m.tw, m.pass);
    double rho = precondition(a, m, turn);
    const double ref = rho;
    double relres = 0.0, pq = 0.0, alpha = 0.0, beta = 0.0;
    int iters = 0, status = FEH_OK;
    bool on = true;
    if (!isfinite(rho)) {
        status = FEH_EBREAKDOWN;
        on = false;
    } else if (!(rho > 0.0)) {
        on = false;
    } else {
        relres = sqrt(rho / ref);
        on = relres > a.tol;
    }
    if (on) {
        inverse<T>(a, m.W, m.tw, m.pass);
        direction<T>(a, m, T(0));
    }
    while (on) {
        pq = all_sum(apply(std::false_type{}), m.red, turn);
        if (!(pq > 0.0) || !isfinite(pq)) {
            status = FEH_EBREAKDOWN;
            break;
        }
        alpha = rho / pq;
        advance(a, m, alpha);
        forward<T>(a, m.W, m.tw, m.pass);
        const double r = precondition(a, m, turn);
        for (int e = threadIdx.x; e < DIM * a.N; e += NT) m.X[e] = fma(U(alpha), U(m.P[e]), m.X[e]);
        ++iters;
        if (!isfinite(r)) {
            status = FEH_EBREAKDOWN;
            break;
        }
        const double rr = r > 0.0 ? r : 0.0;
        relres = sqrt(rr / ref);
        if (relres <= a.tol) break;
        if (iters >= a.max_iter) {
            status = FEH_ENOCONV;
            break;
        }
        beta = rr / rho;
        rho = rr;
        inverse<T>(a, m.W, m.tw, m.pass);
        direction<T>(a, m, T(beta));
    }
    for (int e = threadIdx.x; e < DIM * a.N; e += NT) static_cast<U *>(a.u)[(long long)l * DIM * a.N + e] = m.X[e];
    if (threadIdx.x == 0) {
        LcState st{};
        st.rho = rho;
        st.rho_ref = ref;
        st.pq = pq;
        st.alpha = alpha;
        st.beta = beta;
        st.relres = relres;
        st.iters = iters;
        st.status = status;
        a.st[l] = st;
    }
}

// Every load step and Newton step of a finite-strain solve (see fs_solve_nodal).
template <typename T, int KIND>
__global__ __launch_bounds__(NT) void k_small_finite(SmallArgs<T> a) {
    static constexpr Stencil s = make_stencil<DIM, KIND>();
    const int l = blockIdx.x;
    const Lds<T, double, true> m(a, 0);
    T *w = reinterpret_cast<T *>(m.W);
    int turn = 0;
    double sc[DIM], Fb[DIM][DIM];
    #pragma unroll
    for (int x = 0; x < DIM; ++x) sc[x] = a.ihd[x] * (s.half ? 0.5 : 1.0);
    // TAN: W = w B^T (K(F) : B p), part of p.q; else W = -w B^T P, part of |P|^2
    auto apply = [&](auto tan) __attribute__((always_inline)) {
        constexpr bool TAN = decltype(tan)::value;
        double acc = 0.0;
        for (int v = threadIdx.x; v < a.N; v += NT) {
            const Place<DIM> pl(a.n, (unsigned)v, a.d_last.div((uint32_t)v));
            double u[32][DIM], q[DIM];
            T p[32][DIM];
            lds_nodes<double>(s, m.F, a.N, pl, u);
            if constexpr (TAN) lds_nodes<T>(s, m.P, a.N, pl, p);
            #pragma unroll
            for (int i = 0; i < DIM; ++i) q[i] = 0.0;
            auto column = [&](int slot, int c, double (&col)[DIM]) __attribute__((always_inline)) {
                const unsigned vo = pl.at(s.vox[slot]);
                T tl, tm;
                material_at(m, vo, tl, tm);
                const double lam = double(tl), mu = double(tm);
                const Grad<DIM> f = add<DIM>(point_grad<DIM, double>(s, slot, u, sc), Fb);
                const double tr = twice_trace<DIM>(f);
                if constexpr (TAN) {
                    const Grad<DIM> x = point_grad<DIM, T>(s, slot, p, sc);
                    double trx = dot<DIM>(f.v[0], x.v[0]);
                    #pragma unroll
                    for (int j = 1; j < DIM; ++j) trx += dot<DIM>(f.v[j], x.v[j]);
                    tangent_column<DIM>(f, x, c, lam, mu, tr, trx, col);
                } else {
                    pk1_column<DIM>(f, c, lam, mu, tr, col);
                }
            };
            #pragma unroll
            for (int k = 0; k < s.nb; ++k) {
                double e[DIM], b[DIM];
                column(s.end[k], s.axis[k], e);
                column(s.start[k], s.axis[k], b);
                #pragma unroll
                for (int i = 0; i < DIM; ++i) q[i] = fma(sc[s.axis[k]], e[i] - b[i], q[i]);
            }
            const int row = (int)a.d_last.div((uint32_t)v), i0 = v - row * a.nlast;
            #pragma unroll
            for (int i = 0; i < DIM; ++i) {
                const T qv = T(TAN ? a.w * q[i] : -a.w * q[i]);
                put_real<T>(a, w, row, i0, i, qv);
                if constexpr (!TAN) m.R[i * a.N + v] = qv;
                if constexpr (TAN) acc += double(p[0][i]) * double(qv);
            }
            if constexpr (!TAN) {
                T tl, tm;
                material_at(m, (unsigned)v, tl, tm);
                const double lam = double(tl), mu = double(tm);
                #pragma unroll
                for (int k = 0; k < s.np; ++k) {
                    const Grad<DIM> f = add<DIM>(point_grad<DIM, double>(s, s.ni + k, u, sc), Fb);
                    const double tr = twice_trace<DIM>(f);
                    #pragma unroll
                    for (int c = 0; c < DIM; ++c) {
                        double col[DIM];
                        pk1_column<DIM>(f, c, lam, mu, tr, col);
                        acc += dot<DIM>(col, col);
                    }
                }
            }
        }
        return acc;
    };
    for (int e = threadIdx.x; e < DIM * a.N; e += NT) m.F[e] = 0.0;
    int newton = 0, cg = 0, status = FEH_OK;
    double rel_eq = 0.0, rel_inc = 0.0;
    for (int step = 1; step <= a.n_steps; ++step) {
        #pragma unroll
        for (int i = 0; i < DIM; ++i)
            #pragma unroll
            for (int j = 0; j < DIM; ++j) {
                const double I = i == j ? 1.0 : 0.0;
                Fb[i][j] = I + (double)step / a.n_steps * (a.Ebar[(l * DIM + i) * DIM + j] - I);
            }
        __syncthreads();
        bool done = false;
        for (int it = 0; it < a.max_newton; ++it) {
            const double nP = sqrt(all_sum(apply(std::false_type{}), m.red, turn));
            forward<T>(a, m.W, m.tw, m.pass);
            double rho = precondition(a, m, turn);
            const double nG = sqrt(rho / a.w);
            rel_eq = nP > 0.0 ? nG / nP : 0.0;
            if (nG <= a.equil_tol * nP) {
                done = true;
                break;
            }
            for (int e = threadIdx.x; e < DIM * a.N; e += NT) m.X[e] = 0.0;
            const double ref = rho;
            bool on = isfinite(rho) && rho > 0.0 && 1.0 > a.tol;
            int iters = 0;
            if (on) {
                inverse<T>(a, m.W, m.tw, m.pass);
                direction<T>(a, m, T(0));
            }
            while (on) {
                const double pq = all_sum(apply(std::true_type{}), m.red, turn);
                if (!(pq > 0.0) || !isfinite(pq)) break;
                const double alpha = rho / pq;
                advance(a, m, alpha);
                forward<T>(a, m.W, m.tw, m.pass);
                const double r = precondition(a, m, turn);
                for (int e = threadIdx.x; e < DIM * a.N; e += NT) m.X[e] = fma(alpha, double(m.P[e]), m.X[e]);
                ++iters;
                if (!isfinite(r)) break;
                const double rr = r > 0.0 ? r : 0.0;
                if (sqrt(rr / ref) <= a.tol || iters >= a.max_iter) break;
                const double beta = rr / rho;
                rho = rr;
                inverse<T>(a, m.W, m.tw, m.pass);
                direction<T>(a, m, T(beta));
            }
            __syncthreads();
            double s1 = 0.0, s2 = 0.0;
            for (int v = threadIdx.x; v < a.N; v += NT) {
                const Place<DIM> pl(a.n, (unsigned)v, a.d_last.div((uint32_t)v));
                double u[32][DIM], d[32][DIM];
                lds_nodes<double>(s, m.F, a.N, pl, u);
                lds_nodes<double>(s, m.X, a.N, pl, d);
                #pragma unroll
                for (int k = 0; k < s.np; ++k) {
                    Grad<DIM> f = add<DIM>(point_grad<DIM, double>(s, s.ni + k, u, sc), Fb);
                    const Grad<DIM> x = point_grad<DIM, double>(s, s.ni + k, d, sc);
                    #pragma unroll
                    for (int c = 0; c < DIM; ++c) {
                        s1 += dot<DIM>(x.v[c], x.v[c]);
                        #pragma unroll
                        for (int i = 0; i < DIM; ++i) f.v[c][i] += x.v[c][i];
                        s2 += dot<DIM>(f.v[c], f.v[c]);
                    }
                }
            }
            const double nd = sqrt(all_sum(s1, m.red, turn)), nf = sqrt(all_sum(s2, m.red, turn));
            for (int e = threadIdx.x; e < DIM * a.N; e += NT) m.F[e] += m.X[e];
            __syncthreads();
            ++newton;
            cg += iters;
            rel_inc = nf > 0.0 ? nd / nf : 0.0;
            if (nd <= a.newton_tol * nf) {
                done = true;
                break;
            }
        }
        if (!done) status = FEH_ENOCONV;
    }
    for (int e = threadIdx.x; e < DIM * a.N; e += NT) a.uf[(long long)l * DIM * a.N + e] = m.F[e];
    if (threadIdx.x < DIM * DIM) a.fbar[l * DIM * DIM + threadIdx.x] = a.Ebar[l * DIM * DIM + threadIdx.x];
    if (threadIdx.x == 0) {
        double *o = a.fin + 5 * l;
        o[0] = newton;
        o[1] = cg;
        o[2] = status;
        o[3] = rel_eq;
        o[4] = rel_inc;
    }
}

// ---------------------------------------------------------------------------
// host
// ---------------------------------------------------------------------------
struct Shape {
    int S;                  // points of a row of W
    size_t lds;             // bytes without what may also stay in global memory
    size_t table, mat;      // of the inverses, of the material
    bool table_in, mat_in;  // kept in LDS as well
    bool fits;
};

template <typename T>
Shape shape_of(const feh_plan &p, bool finite) {
    Shape h{};
    const long long nlast = p.n[DIM - 1], rows = p.N / nlast;
    h.S = (int)(p.last_even ? p.nh : nlast);
    auto up = [](size_t b) { return (b + 15) & ~size_t(15); };
    const size_t points = (size_t)rows * h.S * DIM, values = (size_t)DIM * p.N;
    h.lds = up(values * sizeof(T)) + up(points * sizeof(Cx<T>)) + up((size_t)DIM * p.Nspec * sizeof(Cx<T>)) +
            up(values * (finite || p.u_f64 ? 8 : sizeof(T))) + up(finite ? values * 8 : 0) + up(2 * NW * 8);
    for (int x = 0; x < DIM; ++x) h.lds += up((size_t)p.n[x] * sizeof(Cx<T>)) + up(5 * kMaxRadixCount * 4);
    h.table = up(4 * (size_t)p.Nspec * sizeof(T));
    h.mat = 2 * up((size_t)p.N * sizeof(T));
    h.mat_in = h.lds + h.mat <= kLdsUse;
    h.table_in = h.lds + (h.mat_in ? h.mat : 0) + h.table <= kLdsUse;
    h.fits = h.lds <= kLdsUse && points <= (size_t)kPoints<T> * NT;
    if (!h.fits) return h;
    for (int x = 0; x < DIM; ++x) {
        const long long batches = x == DIM - 1 ? rows * DIM : p.Nspec / p.n[x] * DIM;
        for (int s = 0; s < p.fft[x].npass; ++s) {
            const int R = p.fft[x].pass[s].R;
            if (R == 2 || R == 3 || R == 4 || R == 5 || R == 8) continue;
            const long long bf = batches * (p.fft[x].n / R);
            const long long tiles = (((R - 1) / 2 + 16) / 16) * ((2 * bf + 15) / 16);
            if (tiles > kTiles * NW) h.fits = false;
        }
    }
    return h;
}

template <typename T>
SmallArgs<T> small_args(const feh_plan &p, const Shape &h) {
    SmallArgs<T> a{};
    for (int x = 0; x < 3; ++x) {
        a.n[x] = (int)p.n[x];
        if (x < DIM) a.tw[x] = p.ptr<const Cx<T>>(p.off_tw[x]);
        a.ih[x] = T(1.0 / p.h[x]);
        a.ihd[x] = 1.0 / p.h[x];
    }
    a.G = p.G;
    a.N = (int)p.N;
    a.nlast = (int)p.n[DIM - 1];
    a.rows = a.N / a.nlast;
    a.even = p.last_even ? 1 : 0;
    a.nc = p.fft[DIM - 1].n;
    a.nh = (int)p.nh;
    a.S = h.S;
    a.nspec = (int)p.Nspec;
    a.inner = (int)(p.Nspec / p.n[0]);
    a.d_N = FastDiv::make((uint32_t)a.N);
    a.d_last = FastDiv::make((uint32_t)a.nlast);
    a.d_nh = FastDiv::make((uint32_t)a.nh);
    a.d_inner = FastDiv::make((uint32_t)a.inner);
    a.d_D = FastDiv::make((uint32_t)DIM);
    a.d_half = FastDiv::make((uint32_t)(a.even ? a.nc / 2 + 1 : a.nh));
    const int lo = a.nh * DIM;
    auto axis = [&](int x, int batches, int lo_, int A, int stride, int tws) {
        a.ax[x].fft = p.fft[x];
        a.ax[x].nb = FastDiv::make((uint32_t)batches);
        a.ax[x].lo = FastDiv::make((uint32_t)lo_);
        a.ax[x].A = A;
        a.ax[x].stride = stride;
        a.ax[x].tws = tws;
    };
    axis(1, a.rows * DIM, DIM, a.S * DIM, DIM, a.even ? 2 : 1);
    axis(0, lo, lo, 0, a.S * DIM, 1);
    a.lam = p.ptr<const T>(p.off_lam);
    a.mu = p.ptr<const T>(p.off_mu);
    a.minv = p.ptr<const T>(p.off_minv);
    a.Ebar = p.ptr<const double>(p.off_ebar);
    a.vol = T(0.5);
    a.invN = 1.0 / (double)p.N;
    a.table_lds = h.table_in ? 1 : 0;
    a.mat_lds = h.mat_in ? 1 : 0;
    return a;
}

template <typename T>
int solve_t(const feh_plan &p, double tol, int max_iter) {
    const Shape h = shape_of<T>(p, false);
    SmallArgs<T> a = small_args<T>(p, h);
    a.u = p.ws + p.off_u;
    a.st = p.ptr<LcState>(p.off_state);
    a.tol = tol;
    a.max_iter = max_iter;
    CK(launch_inverse_table(p));
    auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(p.L), dim3(NT), h.lds + (h.table_in ? h.table : 0) + (h.mat_in ? h.mat : 0), p.stream, a);
    };
    if (p.u_f64) run(k_small_solve<T, double>);
    else run(k_small_solve<T, T>);
    return hip_check(hipGetLastError(), "one-workgroup solve");
}

template <typename T>
int finite_t(const feh_plan &p, int kind, const SmallFinite &f) {
    const Shape h = shape_of<T>(p, true);
    SmallArgs<T> a = small_args<T>(p, h);
    a.Ebar = f.Fbar_end;
    a.fbar = f.fbar;
    a.uf = f.u;
    a.fin = f.out;
    a.w = kind == FEH_DERIV_FE ? 0.5 : 1.0;
    a.tol = f.cg_tol;
    a.max_iter = f.max_cg;
    a.n_steps = f.n_steps;
    a.max_newton = f.max_newton;
    a.newton_tol = f.newton_tol;
    a.equil_tol = f.equil_tol;
    CK(launch_inverse_table(p));
    auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(p.L), dim3(NT), h.lds + (h.table_in ? h.table : 0) + (h.mat_in ? h.mat : 0), p.stream, a);
    };
    switch (kind) {
    case FEH_DERIV_FE: run(k_small_finite<T, FEH_DERIV_FE>); break;
    case FEH_DERIV_FD: run(k_small_finite<T, FEH_DERIV_FD>); break;
    case FEH_DERIV_CD: run(k_small_finite<T, FEH_DERIV_CD>); break;
    default: run(k_small_finite<T, FEH_DERIV_LS>); break;
    }
    return hip_check(hipGetLastError(), "one-workgroup finite strain");
}

}  // namespace

// A plan that is being profiled runs the passes it asks about.
bool small_solve_ok(const feh_plan &p, bool finite) {
    if (p.dim != DIM || p.tune_general || p.prof_on) return false;
    return p.prec == FEH_FP64 ? shape_of<double>(p, finite).fits : shape_of<float>(p, finite).fits;
}

int launch_small_solve(const feh_plan &p, double tol, int max_iter) {
    return p.prec == FEH_FP64 ? solve_t<double>(p, tol, max_iter) : solve_t<float>(p, tol, max_iter);
}

int launch_small_finite(const feh_plan &p, int kind, const SmallFinite &f) {
    return p.prec == FEH_FP64 ? finite_t<double>(p, kind, f) : finite_t<float>(p, kind, f);
}

}  // namespace feh
