// Operators of the stencil derivatives on nodal fields: B^T P(B u), its
// tangent, and the point sums of the finite-strain solver, with the
// deformation gradient formed from u where it is used.
//
// A stencil derivative (linear finite elements, forward and central
// differences, least squares) gives at each evaluation point T of a voxel
// the gradient g_ia = d u_i / d x_a as differences of a nodal field, so a
// compatible field is B u of D values a node, whatever the n_e D^2 (finite
// strain: 54 in 3D FE) components of the field itself.  B and B^T are applied
// here as a gather: one thread owns a node, evaluates every point that the
// node's value enters (24 tetrahedra in 3D FE, 6 triangles in 2D FE) and sums
// the columns of P that pull on it.  Points are evaluated once per node they
// touch (4 times in 3D FE), but the point itself keeps nothing in memory and
// no two threads exchange anything: no LDS, no barrier, one kernel for every
// kind, and only the columns of P that the node needs are formed.  All
// arithmetic is FP64 (its rate is that of non-packed FP32 on this chip); u is
// read in double, the search direction in the plan precision.
//
// The columns are summed in brackets, the column at one end of an edge less
// the same edge's column one voxel on: near equilibrium the two nearly cancel
// and their difference is exact, so the force has the rounding of its own
// size, not of P's.  (Summed one by one, the residual of a pillar separated by
// vacuum kept a resultant of 1e-16 |P| that no deformation balances, and CG on
// a late Newton step diverged on it.)  That needs a point's column to be the
// same number for every node that forms it: products and sums are written as
// fma or kept apart (no contraction), never left to the compiler.
// Bound: FP64 arithmetic in 3D (about 2000 operations a node for the tangent).
#include <algorithm>

#include "device_common.hpp"

#pragma clang fp contract(off)

namespace feh {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxBlocks = 8192;  // partial sums a load case

// ---------------------------------------------------------------------------
// The stencils as tables, built at compile time: the nodes (offsets from the
// thread's node) that are read; the points the node enters, each with its
// voxel and, per axis a, up to two edges (plus, minus node) whose sum
// (times 1/2 for two) is h_a g_ia; the points of the node's own voxel; and the
// brackets: column a of P at the point whose edge ends at the node less that
// of the same edge of the voxel it starts from.
// ---------------------------------------------------------------------------
struct Stencil {
    int nn = 0, node[32][3] = {};
    int ni = 0, np = 0;
    int vox[24][3] = {}, type[24] = {};        // voxel and point of an incident slot
    int plus[30][3][2] = {}, minus[30][3][2] = {};  // incident points, then own points
    int nb = 0, axis[18] = {}, end[18] = {}, start[18] = {};
    bool half = false, two = false;            // edges carry 1/2; two edges an axis

    constexpr int at(int x, int y, int z) {
        for (int i = 0; i < nn; ++i)
            if (node[i][0] == x && node[i][1] == y && node[i][2] == z) return i;
        node[nn][0] = x;
        node[nn][1] = y;
        node[nn][2] = z;
        return nn++;
    }
};

struct Edge {
    int m[3], p[3];
};

// edges e[a][0..1] of a point of the voxel at v, relative to the voxel
template <int DIM>
constexpr void put_point(Stencil &s, int slot, const int (&v)[3], const Edge (&e)[3][2]) {
    for (int a = 0; a < DIM; ++a)
        for (int k = 0; k < (s.two ? 2 : 1); ++k) {
            s.plus[slot][a][k] = s.at(v[0] + e[a][k].p[0], v[1] + e[a][k].p[1], v[2] + e[a][k].p[2]);
            s.minus[slot][a][k] = s.at(v[0] + e[a][k].m[0], v[1] + e[a][k].m[1], v[2] + e[a][k].m[2]);
        }
}

// edges of point t of the voxel at the origin
template <int DIM, int KIND>
constexpr void point_edges(int t, Edge (&e)[3][2]) {
    for (int a = 0; a < 3; ++a)
        for (int k = 0; k < 2; ++k) e[a][k] = Edge{};
    if constexpr (KIND == FEH_DERIV_FE && DIM == 3) {
        constexpr int P[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
        int c[3] = {0, 0, 0};
        for (int j = 0; j < 3; ++j) {
            const int a = P[t][j];
            for (int b = 0; b < 3; ++b) e[a][0].m[b] = c[b];
            c[a] = 1;
            for (int b = 0; b < 3; ++b) e[a][0].p[b] = c[b];
        }
    } else if constexpr (KIND == FEH_DERIV_FE) {
        // triangle 0: 00 -> 10, 00 -> 01; triangle 1: 01 -> 11, 10 -> 11
        for (int a = 0; a < 2; ++a) {
            e[a][0].p[a] = 1;
            if (t == 1) e[a][0].m[1 - a] = e[a][0].p[1 - a] = 1;
        }
    } else if constexpr (KIND == FEH_DERIV_FD) {
        for (int a = 0; a < DIM; ++a) e[a][0].p[a] = 1;
    } else if constexpr (KIND == FEH_DERIV_CD) {
        for (int a = 0; a < DIM; ++a) {
            e[a][0].p[a] = 1;
            e[a][0].m[a] = -1;
        }
    } else {  // least squares, 2D: the mean of the two edges along each axis
        for (int a = 0; a < 2; ++a)
            for (int k = 0; k < 2; ++k) {
                e[a][k].p[a] = 1;
                e[a][k].m[1 - a] = e[a][k].p[1 - a] = k;
            }
    }
}

// slot of point t of the voxel at v, added when it is new
template <int DIM, int KIND>
constexpr int incident(Stencil &s, int t, const int (&v)[3]) {
    for (int k = 0; k < s.ni; ++k)
        if (s.type[k] == t && s.vox[k][0] == v[0] && s.vox[k][1] == v[1] && s.vox[k][2] == v[2]) return k;
    Edge e[3][2] = {};
    point_edges<DIM, KIND>(t, e);
    put_point<DIM>(s, s.ni, v, e);
    s.type[s.ni] = t;
    for (int a = 0; a < 3; ++a) s.vox[s.ni][a] = v[a];
    return s.ni++;
}

template <int DIM, int KIND>
constexpr Stencil make_stencil() {
    Stencil s;
    s.half = KIND == FEH_DERIV_CD || KIND == FEH_DERIV_LS;
    s.two = KIND == FEH_DERIV_LS;
    s.np = KIND == FEH_DERIV_FE ? (DIM == 3 ? 6 : 2) : 1;
    s.at(0, 0, 0);
    for (int t = 0; t < s.np; ++t) {
        Edge e[3][2] = {};
        point_edges<DIM, KIND>(t, e);
        for (int a = 0; a < DIM; ++a)
            for (int k = 0; k < (s.two ? 2 : 1); ++k) {
                const int ve[3] = {-e[a][k].p[0], -e[a][k].p[1], -e[a][k].p[2]};
                const int vs[3] = {-e[a][k].m[0], -e[a][k].m[1], -e[a][k].m[2]};
                s.axis[s.nb] = a;
                s.end[s.nb] = incident<DIM, KIND>(s, t, ve);
                s.start[s.nb] = incident<DIM, KIND>(s, t, vs);
                ++s.nb;
            }
    }
    const int o[3] = {0, 0, 0};
    for (int t = 0; t < s.np; ++t) {
        Edge e[3][2] = {};
        point_edges<DIM, KIND>(t, e);
        put_point<DIM>(s, s.ni + t, o, e);
    }
    return s;
}

template <typename T>
struct NK {
    const double *u;       // [L][D][N]
    const T *p;            // tangent: search direction; norms: unused
    const double *du;      // norms: increment
    T *out;                // [L][D][N]
    T *Fout, *Pout;        // post: [L][N][n_e][D][D]
    const T *lam, *mu;
    const double *Fbar;    // [L][D][D]
    double *partial;       // [L][stride] (or [quantity][blocks])
    const LcState *st;
    const int *mask;
    long long N;
    int n[3];
    int L, nblk, stride;
    double ih[3], w;       // 1 / h_a; weight of a point
};

// columns g[a][i] = d u_i / d x_a of a point, from the nodes' values
template <int DIM>
struct Grad {
    double v[DIM][DIM];
};

template <int DIM, typename V>
__device__ __forceinline__ Grad<DIM> point_grad(const Stencil &s, int slot, const V (&u)[32][DIM], const double (&sc)[DIM]) {
    Grad<DIM> g;
    #pragma unroll
    for (int a = 0; a < DIM; ++a)
        #pragma unroll
        for (int i = 0; i < DIM; ++i) {
            double d = double(u[s.plus[slot][a][0]][i]) - double(u[s.minus[slot][a][0]][i]);
            if (s.two) d += double(u[s.plus[slot][a][1]][i]) - double(u[s.minus[slot][a][1]][i]);
            g.v[a][i] = d * sc[a];
        }
    return g;
}

template <int DIM>
__device__ __forceinline__ double dot(const double (&x)[DIM], const double (&y)[DIM]) {
    double s = x[0] * y[0];
    #pragma unroll
    for (int i = 1; i < DIM; ++i) s = fma(x[i], y[i], s);
    return s;
}

// Saint Venant-Kirchhoff: column a of P = F (lam tr(E) I + 2 mu E), with
// E_ja = (F_j . F_a - delta_ja) / 2 of the columns F_j; tr = 2 tr(E).
template <int DIM>
__device__ __forceinline__ double twice_trace(const Grad<DIM> &f) {
    double t = -double(DIM);
    #pragma unroll
    for (int j = 0; j < DIM; ++j) t += dot<DIM>(f.v[j], f.v[j]);
    return t;
}
template <int DIM>
__device__ __forceinline__ void pk1_column(const Grad<DIM> &f, int a, double lam, double mu, double tr, double (&c)[DIM]) {
    double s[DIM];
    #pragma unroll
    for (int j = 0; j < DIM; ++j) s[j] = mu * (dot<DIM>(f.v[j], f.v[a]) - (j == a ? 1.0 : 0.0));
    s[a] += 0.5 * lam * tr;
    #pragma unroll
    for (int i = 0; i < DIM; ++i) {
        c[i] = f.v[0][i] * s[0];
        #pragma unroll
        for (int j = 1; j < DIM; ++j) c[i] = fma(f.v[j][i], s[j], c[i]);
    }
}
// column a of dP = X S + F dS, dS = lam tr(dE) I + 2 mu dE, dE = sym(F^T X);
// trx = tr(dE) = sum_j F_j . X_j
template <int DIM>
__device__ __forceinline__ void tangent_column(const Grad<DIM> &f, const Grad<DIM> &x, int a, double lam, double mu,
                                               double tr, double trx, double (&c)[DIM]) {
    double s[DIM], d[DIM];
    #pragma unroll
    for (int j = 0; j < DIM; ++j) {
        s[j] = mu * (dot<DIM>(f.v[j], f.v[a]) - (j == a ? 1.0 : 0.0));
        d[j] = mu * (dot<DIM>(f.v[j], x.v[a]) + dot<DIM>(x.v[j], f.v[a]));
    }
    s[a] += 0.5 * lam * tr;
    d[a] += lam * trx;
    #pragma unroll
    for (int i = 0; i < DIM; ++i) {
        c[i] = x.v[0][i] * s[0];
        #pragma unroll
        for (int j = 0; j < DIM; ++j) {
            if (j > 0) c[i] = fma(x.v[j][i], s[j], c[i]);
            c[i] = fma(f.v[j][i], d[j], c[i]);
        }
    }
}

// Offsets of the stencil's nodes from the load case's component base, and of
// the incident points' voxels.
template <int DIM>
struct Place {
    unsigned o[3][5];  // wrapped axis offsets at -2 .. 2, scaled by the axis stride
    __device__ __forceinline__ Place(const int (&n)[3], unsigned v) {
        int c[3] = {0, 0, 0};
        const unsigned last = (unsigned)n[DIM - 1];
        const unsigned r = v / last;
        c[DIM - 1] = (int)(v - r * last);
        if constexpr (DIM == 3) {
            c[0] = (int)(r / (unsigned)n[1]);
            c[1] = (int)(r - (unsigned)c[0] * (unsigned)n[1]);
        } else {
            c[0] = (int)r;
        }
        unsigned st = 1;
        #pragma unroll
        for (int a = DIM - 1; a >= 0; --a) {
            #pragma unroll
            for (int d = -2; d <= 2; ++d) o[a][d + 2] = (unsigned)wrap(c[a] + d, n[a]) * st;
            st *= (unsigned)n[a];
        }
    }
    __device__ __forceinline__ unsigned at(const int (&d)[3]) const {
        unsigned r = o[0][d[0] + 2] + o[1][d[1] + 2];
        if constexpr (DIM == 3) r += o[2][d[2] + 2];
        return r;
    }
};

template <int DIM, typename V>
__device__ __forceinline__ void load_nodes(const Stencil &s, const V *f, long long N, const Place<DIM> &pl, int count,
                                           V (&u)[32][DIM]) {
    #pragma unroll
    for (int i = 0; i < 32; ++i) {
        if (i >= count) break;
        const unsigned o = pl.at(s.node[i]);
        #pragma unroll
        for (int c = 0; c < DIM; ++c) u[i][c] = f[(long long)c * N + o];
    }
}

template <int DIM>
__device__ __forceinline__ Grad<DIM> add(const Grad<DIM> &g, const double (&Fb)[DIM][DIM]) {
    Grad<DIM> r;
    #pragma unroll
    for (int a = 0; a < DIM; ++a)
        #pragma unroll
        for (int i = 0; i < DIM; ++i) r.v[a][i] = g.v[a][i] + Fb[i][a];
    return r;
}

template <typename T, int DIM>
__device__ __forceinline__ void consts(const NK<T> &a, const Stencil &s, int l, double (&sc)[DIM], double (&Fb)[DIM][DIM]) {
    #pragma unroll
    for (int x = 0; x < DIM; ++x) sc[x] = a.ih[x] * (s.half ? 0.5 : 1.0);
    #pragma unroll
    for (int i = 0; i < DIM; ++i)
        #pragma unroll
        for (int j = 0; j < DIM; ++j) Fb[i][j] = a.Fbar[(l * DIM + i) * DIM + j];
}

// TAN: out = w B^T (K(F) : B p) with the partial of p . out, for the active
// load cases; else out = -w B^T P(F) with the partial of the own points' |P|^2.
template <typename T, int DIM, int KIND, bool TAN>
__global__ __launch_bounds__(kThreads) void k_nodal(NK<T> a) {
    static constexpr Stencil s = make_stencil<DIM, KIND>();
    __shared__ double red[kThreads / 64];
    const int t = xcd_remap(blockIdx.x, a.nblk * a.L);
    const int l = t / a.nblk, blk = t - l * a.nblk;
    if (TAN && !a.st[l].active) return;
    double sc[DIM], Fb[DIM][DIM];
    consts<T, DIM>(a, s, l, sc, Fb);
    const long long base = (long long)l * DIM * a.N;
    double acc = 0.0;
    for (long long v = blk * (long long)kThreads + threadIdx.x; v < a.N; v += (long long)a.nblk * kThreads) {
        const Place<DIM> pl(a.n, (unsigned)v);
        double u[32][DIM];
        T p[32][DIM];
        load_nodes<DIM, double>(s, a.u + base, a.N, pl, s.nn, u);
        if constexpr (TAN) load_nodes<DIM, T>(s, a.p + base, a.N, pl, s.nn, p);
        double q[DIM];
        #pragma unroll
        for (int i = 0; i < DIM; ++i) q[i] = 0.0;
        // column c of P (or of dP) at the incident point `slot`
        auto column = [&](int slot, int c, double (&col)[DIM]) __attribute__((always_inline)) {
            const unsigned vo = pl.at(s.vox[slot]);
            const double lam = double(a.lam[vo]), mu = double(a.mu[vo]);
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
        #pragma unroll
        for (int i = 0; i < DIM; ++i) {
            const T qv = T(TAN ? a.w * q[i] : -a.w * q[i]);
            a.out[base + (long long)i * a.N + v] = qv;
            if constexpr (TAN) acc += double(p[0][i]) * double(qv);
        }
        if constexpr (!TAN) {
            const double lam = double(a.lam[v]), mu = double(a.mu[v]);
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
    const double tot = block_sum<kThreads>(acc, red);
    if (threadIdx.x == 0) a.partial[(long long)l * a.stride + blk] = tot;
}

// Partials of |B du|^2 (masked load cases: 0) and of |F|^2 after the step
// F = Fbar + B (u + du), in two arrays of L rows.
template <typename T, int DIM, int KIND>
__global__ __launch_bounds__(kThreads) void k_nodal_norms(NK<T> a) {
    static constexpr Stencil s = make_stencil<DIM, KIND>();
    __shared__ double red[kThreads / 64];
    const int l = blockIdx.y;
    double sc[DIM], Fb[DIM][DIM];
    consts<T, DIM>(a, s, l, sc, Fb);
    const bool on = a.mask[l] != 0;
    const long long base = (long long)l * DIM * a.N;
    double s1 = 0.0, s2 = 0.0;
    for (long long v = blockIdx.x * (long long)kThreads + threadIdx.x; v < a.N; v += (long long)gridDim.x * kThreads) {
        const Place<DIM> pl(a.n, (unsigned)v);
        double u[32][DIM], d[32][DIM];
        load_nodes<DIM, double>(s, a.u + base, a.N, pl, s.nn, u);
        if (on) load_nodes<DIM, double>(s, a.du + base, a.N, pl, s.nn, d);
        #pragma unroll
        for (int k = 0; k < s.np; ++k) {
            Grad<DIM> f = add<DIM>(point_grad<DIM, double>(s, s.ni + k, u, sc), Fb);
            if (on) {
                const Grad<DIM> x = point_grad<DIM, double>(s, s.ni + k, d, sc);
                #pragma unroll
                for (int c = 0; c < DIM; ++c) {
                    s1 += dot<DIM>(x.v[c], x.v[c]);
                    #pragma unroll
                    for (int i = 0; i < DIM; ++i) f.v[c][i] += x.v[c][i];
                }
            }
            #pragma unroll
            for (int c = 0; c < DIM; ++c) s2 += dot<DIM>(f.v[c], f.v[c]);
        }
    }
    const double t1 = block_sum<kThreads>(s1, red);
    const double t2 = block_sum<kThreads>(s2, red);
    if (threadIdx.x == 0) {
        a.partial[(long long)l * a.stride + blockIdx.x] = t1;
        a.partial[(long long)(a.L + l) * a.stride + blockIdx.x] = t2;
    }
}

// u += du of the masked load cases
__global__ __launch_bounds__(kThreads) void k_nodal_add(double *u, const double *du, const int *mask, long long per) {
    const int l = blockIdx.y;
    if (!mask[l]) return;
    for (long long i = blockIdx.x * (long long)kThreads + threadIdx.x; i < per; i += (long long)gridDim.x * kThreads)
        u[l * per + i] += du[l * per + i];
}

// Sums of P over the points (quantity l D^2 + i D + c) and the F and P fields.
template <typename T, int DIM, int KIND>
__global__ __launch_bounds__(kThreads) void k_nodal_post(NK<T> a) {
    static constexpr Stencil s = make_stencil<DIM, KIND>();
    __shared__ double red[kThreads / 64];
    const int l = blockIdx.y;
    double sc[DIM], Fb[DIM][DIM];
    consts<T, DIM>(a, s, l, sc, Fb);
    const long long base = (long long)l * DIM * a.N;
    double sum[DIM][DIM] = {};
    for (long long v = blockIdx.x * (long long)kThreads + threadIdx.x; v < a.N; v += (long long)gridDim.x * kThreads) {
        const Place<DIM> pl(a.n, (unsigned)v);
        double u[32][DIM];
        load_nodes<DIM, double>(s, a.u + base, a.N, pl, s.nn, u);
        const double lam = double(a.lam[v]), mu = double(a.mu[v]);
        #pragma unroll
        for (int k = 0; k < s.np; ++k) {
            const Grad<DIM> f = add<DIM>(point_grad<DIM, double>(s, s.ni + k, u, sc), Fb);
            const double tr = twice_trace<DIM>(f);
            const long long o = (((long long)l * a.N + v) * s.np + k) * DIM * DIM;
            #pragma unroll
            for (int c = 0; c < DIM; ++c) {
                double col[DIM];
                pk1_column<DIM>(f, c, lam, mu, tr, col);
                #pragma unroll
                for (int i = 0; i < DIM; ++i) {
                    sum[i][c] += col[i];
                    if (a.Fout) a.Fout[o + i * DIM + c] = T(f.v[c][i]);
                    if (a.Pout) a.Pout[o + i * DIM + c] = T(col[i]);
                }
            }
        }
    }
    #pragma unroll
    for (int i = 0; i < DIM; ++i)
        #pragma unroll
        for (int c = 0; c < DIM; ++c) {
            const double t = block_sum<kThreads>(sum[i][c], red);
            if (threadIdx.x == 0) a.partial[(long long)((l * DIM + i) * DIM + c) * a.stride + blockIdx.x] = t;
        }
}

__global__ __launch_bounds__(kThreads) void k_nodal_reduce(const double *part, int nblk, int stride, double *out, double scale) {
    __shared__ double red[kThreads / 64];
    double v = 0.0;
    for (int i = threadIdx.x; i < nblk; i += kThreads) v += part[(long long)blockIdx.x * stride + i];
    const double s = block_sum<kThreads>(v, red);
    if (threadIdx.x == 0) out[blockIdx.x] = s * scale;
}

template <typename T>
NK<T> args(const feh_plan &p, const NodalOp &op) {
    NK<T> a{};
    a.u = op.u;
    a.lam = p.ptr<const T>(p.off_lam);
    a.mu = p.ptr<const T>(p.off_mu);
    a.Fbar = op.Fbar;
    a.N = p.N;
    for (int x = 0; x < 3; ++x) {
        a.n[x] = (int)p.n[x];
        a.ih[x] = 1.0 / p.h[x];
    }
    a.L = p.L;
    a.nblk = nodal_num_parts(p);
    a.stride = (int)p.part_stride;
    a.w = 1.0 / (op.kind == FEH_DERIV_FE ? (p.dim == 3 ? 6.0 : 2.0) : 1.0);
    a.partial = op.partial;
    return a;
}

enum What { W_TANGENT, W_RESIDUAL, W_NORMS, W_POST };

template <typename T, int DIM, int KIND>
void go(const feh_plan &p, const NK<T> &a, int what) {
    const dim3 g(a.nblk * a.L), g2(a.nblk, a.L), b(kThreads);
    if (what == W_TANGENT) hipLaunchKernelGGL((k_nodal<T, DIM, KIND, true>), g, b, 0, p.stream, a);
    else if (what == W_RESIDUAL) hipLaunchKernelGGL((k_nodal<T, DIM, KIND, false>), g, b, 0, p.stream, a);
    else if (what == W_NORMS) hipLaunchKernelGGL((k_nodal_norms<T, DIM, KIND>), g2, b, 0, p.stream, a);
    else hipLaunchKernelGGL((k_nodal_post<T, DIM, KIND>), g2, b, 0, p.stream, a);
}

template <typename T>
int dispatch(const feh_plan &p, const NK<T> &a, int kind, int what) {
    if (p.dim == 3) {
        switch (kind) {
        case FEH_DERIV_FE: go<T, 3, FEH_DERIV_FE>(p, a, what); break;
        case FEH_DERIV_FD: go<T, 3, FEH_DERIV_FD>(p, a, what); break;
        case FEH_DERIV_CD: go<T, 3, FEH_DERIV_CD>(p, a, what); break;
        default: return set_error(FEH_ENOTSUP, "derivative kind without a nodal stencil");
        }
    } else {
        switch (kind) {
        case FEH_DERIV_FE: go<T, 2, FEH_DERIV_FE>(p, a, what); break;
        case FEH_DERIV_FD: go<T, 2, FEH_DERIV_FD>(p, a, what); break;
        case FEH_DERIV_CD: go<T, 2, FEH_DERIV_CD>(p, a, what); break;
        case FEH_DERIV_LS: go<T, 2, FEH_DERIV_LS>(p, a, what); break;
        default: return set_error(FEH_ENOTSUP, "derivative kind without a nodal stencil");
        }
    }
    return hip_check(hipGetLastError(), "nodal operator");
}

}  // namespace

bool nodal_kind(int kind, int dim) {
    return kind == FEH_DERIV_FE || kind == FEH_DERIV_FD || kind == FEH_DERIV_CD || (kind == FEH_DERIV_LS && dim == 2);
}

int nodal_num_parts(const feh_plan &p) {
    return (int)std::min<long long>((p.N + kThreads - 1) / kThreads, kMaxBlocks);
}

int launch_nodal_tangent(const feh_plan &p, const NodalOp &op, const void *pv, void *q, const LcState *st) {
    auto run = [&](auto tag) {
        using T = decltype(tag);
        NK<T> a = args<T>(p, op);
        a.p = static_cast<const T *>(pv);
        a.out = static_cast<T *>(q);
        a.st = st;
        return dispatch<T>(p, a, op.kind, W_TANGENT);
    };
    return p.prec == FEH_FP64 ? run(double{}) : run(float{});
}

int launch_nodal_residual(const feh_plan &p, const NodalOp &op, void *r) {
    auto run = [&](auto tag) {
        using T = decltype(tag);
        NK<T> a = args<T>(p, op);
        a.out = static_cast<T *>(r);
        return dispatch<T>(p, a, op.kind, W_RESIDUAL);
    };
    return p.prec == FEH_FP64 ? run(double{}) : run(float{});
}

int launch_nodal_step(const feh_plan &p, const NodalOp &op, double *u, const double *du, const int *mask) {
    auto run = [&](auto tag) {
        using T = decltype(tag);
        NK<T> a = args<T>(p, op);
        a.du = du;
        a.mask = mask;
        return dispatch<T>(p, a, op.kind, W_NORMS);
    };
    CK(p.prec == FEH_FP64 ? run(double{}) : run(float{}));
    const long long per = p.N * p.dim;
    hipLaunchKernelGGL(k_nodal_add, dim3((unsigned)std::min<long long>((per + kThreads - 1) / kThreads, kMaxBlocks), p.L),
                       dim3(kThreads), 0, p.stream, u, du, mask, per);
    return hip_check(hipGetLastError(), "nodal update");
}

int launch_nodal_post(const feh_plan &p, const NodalOp &op, void *F, void *P) {
    auto run = [&](auto tag) {
        using T = decltype(tag);
        NK<T> a = args<T>(p, op);
        a.Fout = static_cast<T *>(F);
        a.Pout = static_cast<T *>(P);
        return dispatch<T>(p, a, op.kind, W_POST);
    };
    return p.prec == FEH_FP64 ? run(double{}) : run(float{});
}

int launch_nodal_reduce(const feh_plan &p, const double *partial, int nq, int nparts, double *out, double scale) {
    hipLaunchKernelGGL(k_nodal_reduce, dim3(nq), dim3(kThreads), 0, p.stream, partial, nparts, (int)p.part_stride, out, scale);
    return hip_check(hipGetLastError(), "nodal reduction");
}

}  // namespace feh
