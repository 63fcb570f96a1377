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
// Bound: FP64 arithmetic in 3D (about 2000 operations a node for the tangent,
// which larger 3D FE grids evaluate once a tetrahedron: nodal_marches()).
#include <algorithm>

#include "nodal_stencil.hpp"

#pragma clang fp contract(off)

namespace feh {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxBlocks = 8192;  // partial sums a load case

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

// Sums of P over the points (quantity l D^2 + i D + c) and the F and P fields,
// whose blocks go through LDS, up to 216 bytes a voxel at a time, so that a
// wavefront writes consecutive values (128^3, 3D FE in FP32: 1170 -> 241 us).
template <typename T, int DIM, int KIND>
__global__ __launch_bounds__(kThreads, 2) void k_nodal_post(NK<T> a) {
    static constexpr Stencil s = make_stencil<DIM, KIND>();
    constexpr int GR = s.np * DIM * DIM * (int)sizeof(T) > 216 ? s.np / 2 : s.np, PER = GR * DIM * DIM;  // points staged together
    static_assert(s.np % GR == 0, "whole groups of points");
    __shared__ T rec[kThreads * PER];
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
        // the wavefront's voxels are consecutive: its first lane's block
        const int lane = (int)threadIdx.x % 64, run = (int)min(64LL, a.N - (v - lane));
        const long long o = ((long long)l * a.N + v - lane) * s.np * DIM * DIM;
        T *row = rec + ((int)threadIdx.x - lane) * PER, *slot = row + lane * PER;
        #pragma unroll
        for (int k0 = 0; k0 < s.np; k0 += GR) {
            // FIELD 0: the sums of P and its field; 1: the field F
            #pragma unroll
            for (int field = 0; field < 2; ++field) {
                T *out = field ? a.Fout : a.Pout;
                if (field && !out) continue;
                #pragma unroll
                for (int k = k0; k < k0 + GR; ++k) {
                    const Grad<DIM> f = add<DIM>(point_grad<DIM, double>(s, s.ni + k, u, sc), Fb);
                    const double tr = twice_trace<DIM>(f);
                    #pragma unroll
                    for (int c = 0; c < DIM; ++c) {
                        double col[DIM];
                        if (!field) pk1_column<DIM>(f, c, lam, mu, tr, col);
                        #pragma unroll
                        for (int i = 0; i < DIM; ++i) {
                            if (!field) sum[i][c] += col[i];
                            if (out) slot[((k - k0) * DIM + i) * DIM + c] = T(field ? f.v[c][i] : col[i]);
                        }
                    }
                }
                if (out) store_run<T, PER, s.np * DIM * DIM>(out + o + k0 * DIM * DIM, row, lane, run);
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

// 3D linear elements: the tangent marches with the edge fluxes exchanged
// through LDS, so that each tetrahedron is evaluated once (and a third again
// on the tiles' borders) where the gather evaluates it for each of its four
// nodes, with 512 registers and so one wave per SIMD besides.  FP32 128^3, one
// load case: 341 -> 132 us.  A march is a chain of planes, though: while every
// node has its own lane on the chip at once (256 CUs x 4 SIMDs x one wave) the
// gather is the faster (whole solves, gather and march: 32^3 2.48 and 2.75 ms,
// 4 x 60 x 200 2.64 and 2.75; beyond it 48^3 3.31 and 3.04, 32^3 x 6 load
// cases 3.94 and 3.60).
bool nodal_marches(const feh_plan &p, int kind) {
    return p.dim == 3 && kind == FEH_DERIV_FE && stencil_rows(p) == 8 && (long long)p.N * p.L > 256 * 4 * 64;
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
