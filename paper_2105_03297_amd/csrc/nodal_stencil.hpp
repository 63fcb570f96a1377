// Stencil derivatives on nodal fields: the tables of a derivative's points and
// the columns of the stress at a point.  Shared by kern_nodal.hip and
// kern_small.hip (internal linkage).  A point's column is the same number for
// every node that forms it: products and sums are written as fma or kept
// apart, never contracted by the compiler.
#pragma once

#include "device_common.hpp"

#pragma clang fp contract(off)

namespace feh {
namespace {

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
    __device__ __forceinline__ Place(const int (&n)[3], unsigned v) : Place(n, v, v / (unsigned)n[DIM - 1]) {}
    // with the row v / n_last
    __device__ __forceinline__ Place(const int (&n)[3], unsigned v, unsigned r) {
        int c[3] = {0, 0, 0};
        c[DIM - 1] = (int)(v - r * (unsigned)n[DIM - 1]);
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

template <int DIM>
__device__ __forceinline__ Grad<DIM> add(const Grad<DIM> &g, const double (&Fb)[DIM][DIM]) {
    Grad<DIM> r;
    #pragma unroll
    for (int a = 0; a < DIM; ++a)
        #pragma unroll
        for (int i = 0; i < DIM; ++i) r.v[a][i] = g.v[a][i] + Fb[i][a];
    return r;
}

}  // namespace
}  // namespace feh
