// Finite-element stencils on the structured grid: q = B^T C B p and friends.
//
// Discretisation (Sec. "Linear finite elements", small-strain appendix): each
// voxel holds n_e linear simplices (2 triangles in 2D, 6 Kuhn tetrahedra in
// 3D) with a constant strain e = sym(grad u) per element, stress
// sigma = lambda tr(e) I + 2 mu e and nodal force |e| B_e^T sigma.
//
// Both B and B^T are written in edge-difference form.  Every element
// gradient is built from differences of nodal values along voxel edges
// (G[:, a] = (u(end) - u(start)) / h_a), so constants map to exactly zero.
// Transposed, every element pushes the column sigma[:, a] |e| / h_a onto the
// voxel edge it used along axis a ("edge flux").  An edge of type (a, c)
// (axis a, start corner c inside its voxel) starting at node n belongs to
// voxel n - c, and the same edge type ending at n to voxel n - e_a - c, so
//   q(n) = sum_{a, c: c_a = 0} [ E_{a,c}(n - e_a - c) - E_{a,c}(n - c) ].
// Each bracket is a difference of the same quantity taken from two voxels:
// in a uniform region every bracket is exactly zero, so a uniform strain in
// a uniform material produces exactly zero force in any precision.
//
// Kernel layout: one workgroup evaluates a VY x VZ tile of voxels in the
// (axis 1, axis 2) plane, one voxel per thread, and marches along axis 0 over
// a chunk of planes.  The nodes it updates are those whose in-plane voxels
// all lie in the tile ((VY - 1) x (VZ - 1) in 3D, VZ - 1 in 2D); neighbouring
// tiles overlap by one voxel row and column, which keeps every wave on the
// same instruction stream (no extra round for halo voxels).  Per step the
// workgroup stages one node plane of the tile (one extra row and column of
// nodes) in LDS, each thread evaluates its voxel (edge fluxes into LDS), and
// each updated node combines the fluxes of its in-plane voxels; the terms
// whose voxels lie in the previous plane are carried in registers (two
// planes per loop trip, so that they alternate between two register sets).
// Global loads and stores go through raw buffers over one plane of one
// component; the lanes that update no node store past the buffer's end,
// which the hardware drops, so the node phase has no branch.  The fused CG
// variant accumulates p.q in FP64 for the step length (the update of p and u
// is fused into the last inverse FFT pass).
#include <algorithm>
#include <type_traits>

#include "device_common.hpp"

namespace feh {
namespace {

// Edge numbering: axis a, start corner c with c_a = 0; k enumerates the
// bits of the two other axes in increasing order (low bit first).
template <int A, int C>
struct EdgeK {
    static constexpr int b = A == 0 ? 1 : 0;
    static constexpr int d = A == 2 ? 1 : 2;
    static constexpr int k = ((C >> b) & 1) | (((C >> d) & 1) << 1);
};

// Strain (+ Ebar) -> stress -> edge fluxes of one tetrahedron with axis path
// (A0, A1, A2), from G[i][a] = d u_i / d x_a.  Eb = (xx, yy, zz, yz, xz, xy).
// E[(a * 4 + k) * 3 + i].  UNIT: all voxel sizes are 1 (no 1/h factors);
// EB: the macroscopic strain enters (right-hand side / residual only).
template <typename T, int A0, int A1, int A2, bool UNIT, bool EB>
__device__ __forceinline__ void tet_edges(const T (&G)[3][3], T lam, T mu, const T (&ih)[3], const T (&Eb)[6],
                                          T (&E)[36]) {
    constexpr int V1 = 1 << A0, V2 = V1 | (1 << A1);
    constexpr int k0 = EdgeK<A0, 0>::k, k1 = EdgeK<A1, V1>::k, k2 = EdgeK<A2, V2>::k;
    T e0 = G[0][0], e1 = G[1][1], e2 = G[2][2];
    if constexpr (EB) {
        e0 += Eb[0];
        e1 += Eb[1];
        e2 += Eb[2];
    }
    const T lt = lam * (e0 + e1 + e2), m2 = mu + mu;
    T S[3][3];
    S[0][0] = lt + m2 * e0;
    S[1][1] = lt + m2 * e1;
    S[2][2] = lt + m2 * e2;
    S[1][2] = S[2][1] = mu * (G[1][2] + G[2][1]);
    S[0][2] = S[2][0] = mu * (G[0][2] + G[2][0]);
    S[0][1] = S[1][0] = mu * (G[0][1] + G[1][0]);
    if constexpr (EB) {
        S[1][2] = S[2][1] = S[1][2] + m2 * Eb[3];
        S[0][2] = S[2][0] = S[0][2] + m2 * Eb[4];
        S[0][1] = S[1][0] = S[0][1] + m2 * Eb[5];
    }
    #pragma unroll
    for (int i = 0; i < 3; ++i) {
        if constexpr (UNIT) {
            E[(A0 * 4 + k0) * 3 + i] += S[i][A0];
            E[(A1 * 4 + k1) * 3 + i] += S[i][A1];
            E[(A2 * 4 + k2) * 3 + i] += S[i][A2];
        } else {
            E[(A0 * 4 + k0) * 3 + i] += S[i][A0] * ih[A0];
            E[(A1 * 4 + k1) * 3 + i] += S[i][A1] * ih[A1];
            E[(A2 * 4 + k2) * 3 + i] += S[i][A2] * ih[A2];
        }
    }
}

template <typename T, int A0, int A1, int A2, bool UNIT, bool EB>
__device__ __forceinline__ void tet_from_nodes(const T (&P)[8][3], T lam, T mu, const T (&ih)[3], const T (&Eb)[6],
                                               T (&E)[36]) {
    constexpr int V1 = 1 << A0, V2 = V1 | (1 << A1);
    T G[3][3];
    #pragma unroll
    for (int i = 0; i < 3; ++i) {
        G[i][A0] = P[V1][i] - P[0][i];
        G[i][A1] = P[V2][i] - P[V1][i];
        G[i][A2] = P[7][i] - P[V2][i];
        if constexpr (!UNIT) {
            G[i][A0] *= ih[A0];
            G[i][A1] *= ih[A1];
            G[i][A2] *= ih[A2];
        }
    }
    tet_edges<T, A0, A1, A2, UNIT, EB>(G, lam, mu, ih, Eb, E);
}

// All six tetrahedra of a voxel; lam, mu already carry the tetrahedron volume.
// The fluxes start at -0: x + (-0) = x exactly for every x (signed zeros
// included), so the first contribution to each edge folds into a move-free
// assignment, which +0 does not allow without relaxed floating-point rules.
template <typename T, bool UNIT, bool EB>
__device__ __forceinline__ void voxel3(const T (&P)[8][3], T lam, T mu, const T (&ih)[3], const T (&Eb)[6],
                                       T (&E)[36]) {
    #pragma unroll
    for (int j = 0; j < 36; ++j) E[j] = T(-0.0);
    tet_from_nodes<T, 0, 1, 2, UNIT, EB>(P, lam, mu, ih, Eb, E);
    tet_from_nodes<T, 0, 2, 1, UNIT, EB>(P, lam, mu, ih, Eb, E);
    tet_from_nodes<T, 1, 0, 2, UNIT, EB>(P, lam, mu, ih, Eb, E);
    tet_from_nodes<T, 1, 2, 0, UNIT, EB>(P, lam, mu, ih, Eb, E);
    tet_from_nodes<T, 2, 0, 1, UNIT, EB>(P, lam, mu, ih, Eb, E);
    tet_from_nodes<T, 2, 1, 0, UNIT, EB>(P, lam, mu, ih, Eb, E);
}

// Finite strain (Saint Venant-Kirchhoff): edge fluxes of dP = X S + F dS of one
// tetrahedron with axis path (A0, A1, A2), F = Fbar + grad u, X = grad p,
// S = lam tr(E) I + 2 mu E, E = (F^T F - I) / 2, dS = lam tr(dE) I + 2 mu dE,
// dE = sym(F^T X), in FP64; Fb[a][i] = Fbar_ia.
// The corner values are read for each tetrahedron anew, by u(c, i) and p(c, i):
// kept for all six, the edge differences alone take 144 registers.
template <int A0, int A1, int A2, bool UNIT, typename FU, typename FP>
__device__ __forceinline__ void tet_tangent(const FU &u, const FP &p, double lam, double mu,
                                            const double (&ih)[3], const double (&Fb)[3][3], double (&E)[36]) {
    asm volatile("" ::: "memory");
    constexpr int V1 = 1 << A0, V2 = V1 | (1 << A1);
    constexpr int k[3] = {EdgeK<A0, 0>::k, EdgeK<A1, V1>::k, EdgeK<A2, V2>::k};
    constexpr int A[3] = {A0, A1, A2}, V[4] = {0, V1, V2, 7};
    double f[3][3], x[3][3];  // columns, by axis
    #pragma unroll
    for (int e = 0; e < 3; ++e)
        #pragma unroll
        for (int i = 0; i < 3; ++i) {
            const double du = u(V[e + 1], i) - u(V[e], i), dp = p(V[e + 1], i) - p(V[e], i);
            f[A[e]][i] = UNIT ? du + Fb[A[e]][i] : fma(du, ih[A[e]], Fb[A[e]][i]);
            x[A[e]][i] = UNIT ? dp : dp * ih[A[e]];
        }
    auto dot = [](const double (&a)[3], const double (&b)[3]) { return fma(a[2], b[2], fma(a[1], b[1], a[0] * b[0])); };
    double s[3][3], d[3][3];
    double tr = -3.0, trx = 0.0;
    #pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double ff = dot(f[a], f[a]), fx = dot(f[a], x[a]);
        tr += ff;
        trx += fx;
        s[a][a] = mu * (ff - 1.0);
        d[a][a] = 2.0 * mu * fx;
    }
    #pragma unroll
    for (int a = 0; a < 3; ++a)
        #pragma unroll
        for (int b = a + 1; b < 3; ++b) {
            s[a][b] = s[b][a] = mu * dot(f[a], f[b]);
            d[a][b] = d[b][a] = mu * (dot(f[a], x[b]) + dot(x[a], f[b]));
        }
    #pragma unroll
    for (int a = 0; a < 3; ++a) {
        s[a][a] = fma(0.5 * lam, tr, s[a][a]);
        d[a][a] = fma(lam, trx, d[a][a]);
    }
    #pragma unroll
    for (int e = 0; e < 3; ++e)
        #pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int a = A[e];
            double c = x[0][i] * s[0][a];
            c = fma(f[0][i], d[0][a], c);
            #pragma unroll
            for (int j = 1; j < 3; ++j) {
                c = fma(x[j][i], s[j][a], c);
                c = fma(f[j][i], d[j][a], c);
            }
            E[(a * 4 + k[e]) * 3 + i] += UNIT ? c : c * ih[a];
        }
}

template <bool UNIT, typename FU, typename FP>
__device__ __forceinline__ void voxel3_tangent(const FU &u, const FP &p, double lam, double mu, const double (&ih)[3],
                                               const double (&Fb)[3][3], double (&E)[36]) {
    #pragma unroll
    for (int j = 0; j < 36; ++j) E[j] = -0.0;
    tet_tangent<0, 1, 2, UNIT>(u, p, lam, mu, ih, Fb, E);
    tet_tangent<0, 2, 1, UNIT>(u, p, lam, mu, ih, Fb, E);
    tet_tangent<1, 0, 2, UNIT>(u, p, lam, mu, ih, Fb, E);
    tet_tangent<1, 2, 0, UNIT>(u, p, lam, mu, ih, Fb, E);
    tet_tangent<2, 0, 1, UNIT>(u, p, lam, mu, ih, Fb, E);
    tet_tangent<2, 1, 0, UNIT>(u, p, lam, mu, ih, Fb, E);
}

// Element field given directly (projection test export): fluxes of |e| sym(e_T).
template <typename T, int A0, int A1, int A2>
__device__ __forceinline__ void tet_div(const T *e, T vol, const T (&ih)[3], T (&E)[36]) {
    constexpr int V1 = 1 << A0, V2 = V1 | (1 << A1);
    constexpr int k0 = EdgeK<A0, 0>::k, k1 = EdgeK<A1, V1>::k, k2 = EdgeK<A2, V2>::k;
    #pragma unroll
    for (int i = 0; i < 3; ++i) {
        E[(A0 * 4 + k0) * 3 + i] += T(0.5) * vol * (e[i * 3 + A0] + e[A0 * 3 + i]) * ih[A0];
        E[(A1 * 4 + k1) * 3 + i] += T(0.5) * vol * (e[i * 3 + A1] + e[A1 * 3 + i]) * ih[A1];
        E[(A2 * 4 + k2) * 3 + i] += T(0.5) * vol * (e[i * 3 + A2] + e[A2 * 3 + i]) * ih[A2];
    }
}

// 2D: element 0 nodes 00,10,01 uses edges (x, c=0) and (y, c=0); element 1
// nodes 11,01,10 uses edges (x, c=e_y) and (y, c=e_x).  Corner index
// c = cx | c1 << 1.  E[(a * 2 + k) * 2 + i], k = offset along the other axis.
template <typename T>
__device__ __forceinline__ void tri_edges(T g00, T g01, T g10, T g11, T lam, T mu, T ihx, T ihy, const T (&Eb)[3],
                                          int kx, int ky, T (&E)[8]) {
    // g_ia = d u_i / d x_a
    const T e0 = g00 + Eb[0], e1 = g11 + Eb[1];
    const T lt = lam * (e0 + e1), m2 = mu + mu;
    const T sxy = mu * (g01 + g10) + m2 * Eb[2];
    E[(0 * 2 + kx) * 2 + 0] = (lt + m2 * e0) * ihx;
    E[(0 * 2 + kx) * 2 + 1] = sxy * ihx;
    E[(1 * 2 + ky) * 2 + 0] = sxy * ihy;
    E[(1 * 2 + ky) * 2 + 1] = (lt + m2 * e1) * ihy;
}

template <typename T>
__device__ __forceinline__ void voxel2(const T (&P)[4][2], T lam, T mu, T ihx, T ihy, const T (&Eb)[3], T (&E)[8]) {
    // element 0: d/dx = (P10 - P00) ihx, d/dy = (P01 - P00) ihy
    tri_edges<T>((P[1][0] - P[0][0]) * ihx, (P[2][0] - P[0][0]) * ihy, (P[1][1] - P[0][1]) * ihx,
                 (P[2][1] - P[0][1]) * ihy, lam, mu, ihx, ihy, Eb, 0, 0, E);
    // element 1: d/dx = (P11 - P01) ihx, d/dy = (P11 - P10) ihy
    tri_edges<T>((P[3][0] - P[2][0]) * ihx, (P[3][0] - P[1][0]) * ihy, (P[3][1] - P[2][1]) * ihx,
                 (P[3][1] - P[1][1]) * ihy, lam, mu, ihx, ihy, Eb, 1, 1, E);
}

template <typename T>
__device__ __forceinline__ void voxel2_div(const T *e, T vol, T ihx, T ihy, T (&E)[8]) {
    // e: [2 elements][2][2]
    #pragma unroll
    for (int el = 0; el < 2; ++el) {
        const T *ee = e + el * 4;
        const T sxy = T(0.5) * vol * (ee[1] + ee[2]);
        E[(0 * 2 + el) * 2 + 0] = vol * ee[0] * ihx;
        E[(0 * 2 + el) * 2 + 1] = sxy * ihx;
        E[(1 * 2 + el) * 2 + 0] = sxy * ihy;
        E[(1 * 2 + el) * 2 + 1] = vol * ee[3] * ihy;
    }
}

template <typename T>
struct SK {
    const T *in0;      // p / u
    T *out0;           // q / r
    const T *lam;
    const T *mu;
    const double *Ebar;
    double *partial;
    const LcState *st;
    int n0, n1, n2;    // 2D: n1 = 1, n2 = n[1]
    long long N;
    int xc, nchunk, nty, ntz, total;
    int part_stride;
    T ih[3];
    T vol;
    const double *u;   // ST_TANGENT: displacement fluctuation
    double ihd[3], vold;
    int ident;         // lambda = 0, mu = 1/2 everywhere
    int G;             // load cases per microstructure (material of load case l: l / G)
};

// Tile shapes: VY x VZ voxels per workgroup (one per thread).  HY = 1 when
// the tile has an axis-1 extent (3D); the node plane of the tile is
// (VY + HY) x (VZ + 1), the updated nodes advance by SY x SZ between tiles.
// 3D tiles are 8 or 16 rows of 32 voxels (256 or 512 threads): the taller
// tile re-reads fewer halo nodes ((VY + 1) 33 loaded per (VY - 1) 31 updated)
// at twice the LDS of the edge-flux exchange.
template <int DIM, int VYT>
struct Tile;
template <int VYT>
struct Tile<3, VYT> {
    static constexpr int VY = VYT, VZ = 32, HY = 1, NC = 3, NEDGE = 12;
    static constexpr int SY = VY - 1, SZ = VZ - 1, NT = VY * VZ;
};
template <int VYT>
struct Tile<2, VYT> {
    static constexpr int VY = 1, VZ = 256, HY = 0, NC = 2, NEDGE = 4;
    static constexpr int SY = 1, SZ = VZ - 1, NT = 256;
};

// The value held by lane - 1 of the wavefront (DPP shift of the whole wave
// right by one lane; lane 0, which has no source lane, receives zero through
// the bound control, so no register has to be zeroed for it).  In the 3D tile
// a row of 32 voxels lies inside one wavefront, so lane - 1 holds the voxel
// at z - 1.
__device__ __forceinline__ int lane_shr1(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xF, 0xF, true); }
__device__ __forceinline__ float from_left(float v) {
    return __builtin_bit_cast(float, lane_shr1(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double from_left(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)lane_shr1((int)(unsigned)b), hi = (unsigned)lane_shr1((int)(unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// TAN (ST_TANGENT, 3D): the finite-strain tangent with the same march, in FP64.
// It keeps u and p of both node planes of a voxel plane in LDS (70 KB, two
// workgroups a CU) and reads them anew for each tetrahedron: with the corners
// in registers as the linear operator has them, 255 registers spilled at two
// waves per SIMD; so none do.  Bound: FP64 arithmetic (128^3: 132 us, of which
// the products and sums are about 60).
template <typename T, int DIM, int MODE, bool UNIT, int VYT>
__global__ __launch_bounds__((Tile<DIM, VYT>::NT)) __attribute__((amdgpu_waves_per_eu(MODE == ST_TANGENT ? 2 : 1))) void k_stencil(SK<T> a) {
    constexpr bool TAN = MODE == ST_TANGENT;
    using CT = std::conditional_t<TAN, double, T>;  // of the fluxes and forces
    using TL = Tile<DIM, VYT>;
    constexpr int VY = TL::VY, VZ = TL::VZ, HY = TL::HY, NC = TL::NC, NEDGE = TL::NEDGE;
    constexpr int EY = VY + HY, EZ = VZ + 1;     // node plane of the tile
    constexpr int NE = EY * EZ, NT = TL::NT;
    constexpr int NQ = NEDGE * NC;               // edge-flux values per voxel
    constexpr int NSE = (NE + NT - 1) / NT;      // node-plane slots per thread
    static_assert(VY * VZ == NT, "one voxel per thread");
    static_assert(DIM == 2 || VZ == 32, "3D: one row of voxels per half wavefront");
    constexpr int NPL = TAN ? 2 : 1;
    __shared__ T Pl[NPL][NC][NE];                // one node plane (TAN: two, in turn)
    // edge fluxes passed through LDS, one column per voxel: in 3D only the 18
    // values the next row of voxels needs (the left neighbour's come by DPP);
    // with the x- and z-edge fluxes raw (24 values) FP64 128^3 x 6 load cases
    // took 309 us, now 289, at 0.9 GB of traffic: bound by the two waves per
    // SIMD that its 200 registers allow (three, at 168, spill: 290)
    constexpr int NX = DIM == 3 ? 18 : NQ;
    __shared__ CT Es[NX][NT];
    __shared__ double Ul[NPL][TAN ? NC : 1][TAN ? NE : 1];  // TAN: the displacement's planes
    __shared__ double red[NT / 64];

    const int tid = threadIdx.x;
    int t = xcd_remap(blockIdx.x, a.total);
    const int tz_t = t % a.ntz;
    t /= a.ntz;
    const int ty_t = t % a.nty;
    t /= a.nty;
    const int ch = t % a.nchunk;
    const int lc = t / a.nchunk;
    const int blk_in_lc = (ch * a.nty + ty_t) * a.ntz + tz_t;

    // load cases that have stopped iterating
    if constexpr (MODE == ST_CG || TAN) {
        if (!a.st[lc].active) return;
    }
    double Fb[3][3] = {};
    if constexpr (TAN) {
        #pragma unroll
        for (int i = 0; i < 3; ++i)
            #pragma unroll
            for (int j = 0; j < 3; ++j) Fb[j][i] = a.Ebar[lc * 9 + 3 * i + j];
    }
    T Eb[6] = {T(0), T(0), T(0), T(0), T(0), T(0)};
    if constexpr (MODE == ST_RESID) {
        const double *E = a.Ebar + lc * DIM * DIM;
        if constexpr (DIM == 3) {
            Eb[0] = T(E[0]); Eb[1] = T(E[4]); Eb[2] = T(E[8]);
            Eb[3] = T(E[5]); Eb[4] = T(E[2]); Eb[5] = T(E[1]);
        } else {
            Eb[0] = T(E[0]); Eb[1] = T(E[3]); Eb[2] = T(E[1]);
        }
    }

    // in-plane origin of the tile's node plane (extended index (0, 0)); the
    // updated nodes start one row (3D) and one column further on
    const int y0 = ty_t * TL::SY - HY, z0 = tz_t * TL::SZ - 1;
    const int x0 = ch * a.xc;
    const int x1 = min(x0 + a.xc, a.n0);
    const long long N = a.N;
    const long long plane = (long long)a.n1 * a.n2;
    const long long lcoff = (long long)lc * NC * N;
    const long long moff = (long long)(lc / a.G) * N;  // this load case's microstructure
    const int ty = tid / VZ, tz = tid - (tid / VZ) * VZ;
    // the thread's voxel has its origin at node (ty, tz) of the tile; that
    // node is updated here when all of its in-plane voxels are in the tile
    const bool owner = ty >= HY && tz >= 1 && y0 + ty < a.n1 && z0 + tz < a.n2;

    // ---- per-thread node slots, fixed for the whole march.  Slot 0 is the
    // thread's own node; later slots cover the last row and column.
    int e_lds[NSE];        // extended node index (an unused slot repeats slot 0)
    unsigned e_boff[NSE];  // in-plane byte offset (the launcher checks that a plane fits 31 bits)
    #pragma unroll
    for (int s = 0; s < NSE; ++s) {
        int ey = -1, ez = -1;
        if (s == 0) {
            ey = ty;
            ez = tz;
        } else {
            const int hh = tid + (s - 1) * NT;  // extra node number
            constexpr int NH = NE - NT;
            if (hh < NH) {
                if constexpr (HY == 0) {
                    ey = 0;  // single row: its last node
                    ez = EZ - 1;
                } else if (hh < EZ) {
                    ey = EY - 1;  // last row
                    ez = hh;
                } else {
                    ey = hh - EZ;  // last column, rows 0 .. EY - 2
                    ez = EZ - 1;
                }
            }
        }
        if (ey >= 0) {
            e_lds[s] = ey * EZ + ez;
            e_boff[s] = (unsigned)(wrap(y0 + ey, a.n1) * a.n2 + wrap(z0 + ez, a.n2)) * (unsigned)sizeof(T);
        } else {
            // unused: its loads re-read the own node and its LDS store
            // repeats the own node's, same value to the same place
            e_lds[s] = e_lds[0];
            e_boff[s] = e_boff[0];
        }
    }
    const long long v_off = (long long)wrap(y0 + ty, a.n1) * a.n2 + wrap(z0 + tz, a.n2);
    const unsigned v_boff = (unsigned)v_off * (unsigned)sizeof(T);
    // node loads and stores go through raw buffers over one plane of one
    // component; a lane that updates no node stores past the buffer's end,
    // which the hardware drops, so no branch splits the node phase
    const unsigned st_boff = owner ? e_boff[0] : 0x80000000u;
    const long long plane_bytes = plane * (long long)sizeof(T);

    // ---- prefetch registers: node plane P and the material of one voxel
    // plane.  Every load is unconditional (unused slots and planes past the
    // chunk re-read valid addresses).
    T rz[NSE][NC];
    double ru[TAN ? NSE : 1][NC];
    T mlam = T(0), mmu = T(0);
    auto fetch_nodes = [&](int P) __attribute__((always_inline)) {
        const long long base = lcoff + (long long)wrap(P, a.n0) * plane;
        #pragma unroll
        for (int s = 0; s < NSE; ++s) {
            #pragma unroll
            for (int c = 0; c < NC; ++c) {
                if constexpr (TAN)
                    ru[s][c] = buffer_ld<double>(raw_buffer(a.u + base + c * N, plane * 8), e_boff[s] * (unsigned)(8 / sizeof(T)));
                if constexpr (MODE == ST_APPLY || MODE == ST_CG || TAN) {
                    rz[s][c] = buffer_ld<T>(raw_buffer(a.in0 + base + c * N, plane_bytes), e_boff[s]);
                } else if constexpr (MODE == ST_RESID) {
                    rz[s][c] = a.in0 ? buffer_ld<T>(raw_buffer(a.in0 + base + c * N, plane_bytes), e_boff[s]) : T(0);
                }
            }
        }
    };
    // stage the fetched node plane in LDS (one plane only: the previous plane's corners
    // stay in registers); returns the thread's own node value in own[]
    T own[NC];
    auto commit_nodes = [&](int w) __attribute__((always_inline)) {
        #pragma unroll
        for (int s = 0; s < NSE; ++s) {
            #pragma unroll
            for (int c = 0; c < NC; ++c) {
                Pl[w][c][e_lds[s]] = rz[s][c];
                if (s == 0) own[c] = rz[s][c];
                if constexpr (TAN) Ul[w][c][e_lds[s]] = ru[s][c];
            }
        }
    };
    auto fetch_material = [&](int V) __attribute__((always_inline)) {
        const long long base = moff + (long long)wrap(V, a.n0) * plane;
        mlam = buffer_ld<T>(raw_buffer(a.lam + base, plane_bytes), v_boff);  // unused (but allocated) for the identity material
        mmu = buffer_ld<T>(raw_buffer(a.mu + base, plane_bytes), v_boff);
    };

    // in-plane corners of the thread's voxel: k = cy + 2 cz (3D), k = cz (2D);
    // Pc holds them in the lower node plane of the current voxel plane
    constexpr int NK = DIM == 3 ? 4 : 2;
    T Pc[NK][NC];
    auto corner_lds = [&](int k) { return DIM == 3 ? (ty + (k & 1)) * EZ + tz + (k >> 1) : tz + k; };

    // carried terms: raw axis-0 edge fluxes of the previous voxel plane, and
    // the differences of the other axes' edges whose voxels lie in the
    // previous plane
    constexpr int NXE = DIM == 3 ? 4 : 2;  // axis-0 edges per voxel
    CT cx[NXE * NC];
    CT cq[NC];
    #pragma unroll
    for (int j = 0; j < NXE * NC; ++j) cx[j] = CT(0);
    #pragma unroll
    for (int c = 0; c < NC; ++c) cq[c] = CT(0);
    double acc = 0.0;

    if constexpr (MODE != ST_DIV) {
        fetch_nodes(x0 - 1);
        commit_nodes(0);
        fetch_nodes(x0);
        __syncthreads();
        #pragma unroll
        for (int k = 0; k < NK; ++k) {
            #pragma unroll
            for (int c = 0; c < NC; ++c) {
                Pc[k][c] = (k == 0) ? own[c] : Pl[0][c][corner_lds(k)];
            }
        }
        __syncthreads();
    }
    fetch_material(x0 - 1);

    // voxel column of the node's in-plane voxels at offset (-dy, -dz); threads
    // that update no node read an interior column instead (results unused)
    const int vo = (ty >= HY && tz >= 1) ? tid : HY * VZ + 1;
    auto vix = [&](int dy, int dz) { return vo - dy * VZ - dz; };

    // one step of the march: the voxels of plane X, then the nodes of plane X
    // (the first step, plane x0 - 1, only primes the carried terms)
    auto step = [&](const int X, auto first, auto buf) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first)::value;
        constexpr int W = TAN ? decltype(buf)::value : 0;  // the LDS plane that takes X + 1
        // ---- stage plane X+1, prefetch plane X+2 and the material of voxel plane X+1
        if constexpr (MODE != ST_DIV) commit_nodes(W);
        const T clam = mlam, cmu = mmu;
        if constexpr (MODE != ST_DIV) fetch_nodes(min(X + 2, x1));
        fetch_material(min(X + 1, x1 - 1));
        __syncthreads();
        // ---- voxel phase: the thread's voxel in plane X
        T pown[NC];  // p at the thread's own node of plane X
        CT q[NC], nq[NC];
        #pragma unroll
        for (int i = 0; i < NC; ++i) {
            q[i] = cq[i];
            nq[i] = CT(-0.0);  // x + (-0) = x: the first term folds into a move
        }
        CT oy[12];   // 3D: the own voxel's axis-1 edge fluxes, kept for the node phase
        {
            T lam, mu;
            if (a.ident) {
                lam = T(0);
                mu = T(0.5) * a.vol;
            } else {
                lam = clam * a.vol;
                mu = cmu * a.vol;
            }
            if constexpr (DIM == 3) {
                CT E[36];
                if constexpr (TAN) {
                    #pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        pown[i] = Pc[0][i];
                        Pc[0][i] = own[i];
                    }
                    auto u = [&](int c, int i) { return Ul[(c & 1) ? W : 1 - W][i][corner_lds(c >> 1)]; };
                    auto pv = [&](int c, int i) { return double(Pl[(c & 1) ? W : 1 - W][i][corner_lds(c >> 1)]); };
                    voxel3_tangent<UNIT>(u, pv, double(clam) * a.vold, double(cmu) * a.vold, a.ihd, Fb, E);
                } else if constexpr (MODE == ST_DIV) {
                    const long long vidx = (long long)wrap(X, a.n0) * plane + v_off;
                    const T *e = a.in0 + ((long long)lc * N + vidx) * 54;
                    #pragma unroll
                    for (int j = 0; j < 36; ++j) E[j] = T(0);
                    tet_div<T, 0, 1, 2>(e + 0, a.vol, a.ih, E);
                    tet_div<T, 0, 2, 1>(e + 9, a.vol, a.ih, E);
                    tet_div<T, 1, 0, 2>(e + 18, a.vol, a.ih, E);
                    tet_div<T, 1, 2, 0>(e + 27, a.vol, a.ih, E);
                    tet_div<T, 2, 0, 1>(e + 36, a.vol, a.ih, E);
                    tet_div<T, 2, 1, 0>(e + 45, a.vol, a.ih, E);
                } else {
                    // corner c = cx + 2 cy + 4 cz; cx = 0 from registers, cx = 1 staged
                    T P[8][3];
                    #pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        #pragma unroll
                        for (int i = 0; i < 3; ++i) {
                            P[2 * k][i] = Pc[k][i];
                            P[2 * k + 1][i] = (k == 0) ? own[i] : Pl[0][i][corner_lds(k)];
                        }
                    }
                    voxel3<T, UNIT, MODE == ST_RESID>(P, lam, mu, a.ih, Eb, E);
                    #pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        #pragma unroll
                        for (int i = 0; i < 3; ++i) {
                            if (k == 0) pown[i] = Pc[0][i];
                            Pc[k][i] = P[2 * k + 1][i];
                        }
                    }
                }
                // terms of the own voxel (x-edge c = 0) and of the left voxel
                // (x-edge c = (0,0,1), z-edges c = (x,0,0) paired with the own voxel),
                // the latter formed by lane - 1, which holds that voxel; and, for
                // the node below, the same of the edges one row on (x-edges
                // c = (0,1,0) and (0,1,1), z-edges c = (x,1,0)), which go to it
                // together with the raw y-edge fluxes: each difference is formed
                // of the two fluxes that nearly cancel, here or there
                #pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const CT c0 = E[0 + i];
                    q[i] += cx[0 * 3 + i] - c0;
                    cx[0 * 3 + i] = c0;
                    const CT c2 = E[6 + i];
                    const CT d2 = cx[2 * 3 + i] - c2;
                    cx[2 * 3 + i] = c2;
                    q[i] += from_left(d2);
                    q[i] += from_left(E[24 + i]) - E[24 + i];
                    nq[i] += from_left(E[27 + i]) - E[27 + i];
                    const CT c1 = E[3 + i];
                    CT below = cx[1 * 3 + i] - c1;
                    cx[1 * 3 + i] = c1;
                    const CT c3 = E[9 + i];
                    const CT d3 = cx[3 * 3 + i] - c3;
                    cx[3 * 3 + i] = c3;
                    below += from_left(d3);
                    below += from_left(E[30 + i]) - E[30 + i];
                    Es[i][tid] = below;
                    Es[3 + i][tid] = from_left(E[33 + i]) - E[33 + i];
                }
                #pragma unroll
                for (int j = 0; j < 12; ++j) {
                    Es[6 + j][tid] = E[12 + j];
                    oy[j] = E[12 + j];
                }
            } else {
                T E[8];
                if constexpr (MODE == ST_DIV) {
                    const long long vidx = (long long)wrap(X, a.n0) * plane + v_off;
                    voxel2_div<T>(a.in0 + ((long long)lc * N + vidx) * 8, a.vol, a.ih[0], a.ih[1], E);
                } else {
                    // corner c = cx + 2 cz
                    T P[4][2];
                    #pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        #pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            P[2 * k][i] = Pc[k][i];
                            P[2 * k + 1][i] = (k == 0) ? own[i] : Pl[0][i][corner_lds(k)];
                        }
                    }
                    const T Eb2[3] = {Eb[0], Eb[1], Eb[2]};
                    voxel2<T>(P, lam, mu, a.ih[0], a.ih[1], Eb2, E);
                    #pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        #pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            if (k == 0) pown[i] = Pc[0][i];
                            Pc[k][i] = P[2 * k + 1][i];
                        }
                    }
                }
                #pragma unroll
                for (int j = 0; j < 8; ++j) Es[j][tid] = E[j];
            }
        }
        __syncthreads();
        // ---- node phase (the thread's own node)
        {
            if constexpr (DIM == 3) {
                // terms of the voxel above (row ty - 1); row 0 reads its own
                // column (it updates no node and feeds no neighbour that does)
                const int ia = ty >= 1 ? tid - VZ : tid;
                CT A[18];
                #pragma unroll
                for (int j = 0; j < 18; ++j) A[j] = Es[j][ia];
                #pragma unroll
                for (int i = 0; i < 3; ++i) {
                    q[i] += A[i];
                    nq[i] += A[3 + i];
                    // y-edges: above - own (k = 0, 1); above-left - left (k = 2, 3) from lane - 1
                    q[i] += A[6 + i] - oy[0 + i];
                    nq[i] += A[9 + i] - oy[3 + i];
                    q[i] += from_left(A[12 + i] - oy[6 + i]);
                    nq[i] += from_left(A[15 + i] - oy[9 + i]);
                }
            } else {
                // axis-0 edges: c = (0, c1), k = c1
                #pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int v = vix(0, k);
                    #pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const T cur = Es[(0 * 2 + k) * 2 + i][v];
                        q[i] += cx[k * 2 + i] - cur;
                        cx[k * 2 + i] = cur;
                    }
                }
                // axis-1 edges: c = (cx, 0), k = cx; voxels n - e_1 - c and n - c
                const int vlo = vix(0, 1), vhi = vix(0, 0);
                #pragma unroll
                for (int i = 0; i < 2; ++i) {
                    q[i] += Es[(1 * 2 + 0) * 2 + i][vlo] - Es[(1 * 2 + 0) * 2 + i][vhi];
                    nq[i] += Es[(1 * 2 + 1) * 2 + i][vlo] - Es[(1 * 2 + 1) * 2 + i][vhi];
                }
            }
            if constexpr (!FIRST) {
                #pragma unroll
                for (int i = 0; i < NC; ++i) {
                    buffer_st<T>(raw_buffer(a.out0 + lcoff + i * N + (long long)X * plane, plane_bytes), st_boff,
                                 MODE == ST_RESID ? T(-q[i]) : T(q[i]));
                    // p.q of every lane (finite values); the lanes that own no
                    // node drop their sum at the end
                    if constexpr (MODE == ST_CG || TAN) acc += double(pown[i]) * double(T(q[i]));
                }
            }
            #pragma unroll
            for (int i = 0; i < NC; ++i) {
                // formed here, next to the lane shifts that feed it, rather
                // than sunk past the march's exit test into the next step
                asm volatile("" : "+v"(nq[i]));
                cq[i] = nq[i];
            }
        }
    };
    // two steps per trip, so that the values carried from one step to the
    // next alternate between two register sets instead of being copied
    using B0 = std::integral_constant<int, 0>;
    using B1 = std::integral_constant<int, 1>;
    step(x0 - 1, std::true_type{}, B1{});
    for (int X = x0;; X += 2) {
        step(X, std::false_type{}, B0{});
        if (X + 1 >= x1) break;
        step(X + 1, std::false_type{}, B1{});
        if (X + 2 >= x1) break;
    }
    if constexpr (MODE == ST_CG || TAN) {
        if (!owner) acc = 0.0;
        const double s = block_sum<NT>(acc, red);
        if (tid == 0) a.partial[(long long)lc * a.part_stride + blk_in_lc] = s;
    }
}

// Planes per workgroup march: 32 in 3D and 8 in 2D (whose rows are short of
// HBM work), where that leaves four workgroups for every CU; a march evaluates
// one plane more than it updates.  With fewer the launch lasts as long as one
// march, and halving it (down to 4 and 2 planes) is the faster: FP32 64^3 x 6
// load cases 46 -> 33 us, 32^3 x 6 38 -> 13, FP64 256^2 x 3 11.7 -> 10.3; at
// 128^3 x 6, which fills the chip, 16 planes are even with 32 and 8 slower
// (163, 163, 173 us).  Counted with 8-row tiles whatever the tile height, and
// no further than the plan's partial sums have room (part_stride; 0 while the
// plan is laid out).
int xchunk(const feh_plan &p) {
    const long long n0 = p.n[0];
    const long long tiles = p.dim == 3 ? ((p.n[1] + 6) / 7) * ((p.n[2] + 30) / 31) : (p.n[1] + 254) / 255;
    int c = p.dim == 3 ? 32 : 8;
    const int least = p.dim == 3 ? 4 : 2;
    while (c > least && (n0 + c - 1) / c * tiles * p.L < 1024 && (n0 + c / 2 - 1) / (c / 2) * tiles <= (long long)p.part_stride)
        c /= 2;
    return (int)std::min<long long>(n0, c);
}

template <typename T, int DIM, int VYT>
int launch_t(const feh_plan &p, int mode, const StencilArgs &sa) {
    using TL = Tile<DIM, VYT>;
    SK<T> a{};
    a.in0 = static_cast<const T *>(sa.in0);
    a.out0 = static_cast<T *>(sa.out0);
    a.lam = p.ptr<const T>(p.off_lam);
    a.mu = p.ptr<const T>(p.off_mu);
    a.Ebar = sa.Ebar;
    a.partial = sa.partial;
    a.st = sa.state;
    a.ident = sa.identity_material ? 1 : 0;
    a.G = p.G;
    a.u = sa.u;
    for (int x = 0; x < 3; ++x) a.ihd[x] = 1.0 / p.h[x];
    a.vold = 1.0 / 6.0;  // ST_TANGENT: the element volume over the voxel's
    if (DIM == 3) {
        a.n0 = (int)p.n[0];
        a.n1 = (int)p.n[1];
        a.n2 = (int)p.n[2];
        a.ih[0] = T(1.0 / p.h[0]);
        a.ih[1] = T(1.0 / p.h[1]);
        a.ih[2] = T(1.0 / p.h[2]);
        a.vol = T(sa.unit_volume ? 1.0 / 6.0 : p.h[0] * p.h[1] * p.h[2] / 6.0);
    } else {
        a.n0 = (int)p.n[0];
        a.n1 = 1;
        a.n2 = (int)p.n[1];
        a.ih[0] = T(1.0 / p.h[0]);
        a.ih[1] = T(1.0 / p.h[1]);
        a.ih[2] = T(1);
        a.vol = T(sa.unit_volume ? 0.5 : p.h[0] * p.h[1] / 2.0);
    }
    // in-plane byte offsets are 32-bit and the store buffers span one plane
    // (at most 4096^2 values: 128 MiB in FP64)
    if ((long long)a.n1 * a.n2 * (long long)sizeof(T) >= (1LL << 31))
        return set_error(FEH_EINVAL, "stencil: one plane of a field must stay below 2 GiB");
    a.N = p.N;
    a.xc = xchunk(p);
    a.nchunk = (a.n0 + a.xc - 1) / a.xc;
    a.nty = (a.n1 + TL::SY - 1) / TL::SY;
    a.ntz = (a.n2 + TL::SZ - 1) / TL::SZ;
    a.total = p.L * a.nchunk * a.nty * a.ntz;
    a.part_stride = (int)p.part_stride;
    dim3 grid(a.total), block(TL::NT);
    const bool unit = p.h[0] == 1.0 && p.h[1] == 1.0 && (DIM == 2 || p.h[2] == 1.0);
#define FEH_STENCIL_CASE(M)                                                                                   \
    case M:                                                                                                   \
        if (unit) hipLaunchKernelGGL((k_stencil<T, DIM, M, true, VYT>), grid, block, 0, p.stream, a);             \
        else hipLaunchKernelGGL((k_stencil<T, DIM, M, false, VYT>), grid, block, 0, p.stream, a);                 \
        break;
    if (mode == ST_TANGENT) {
        if constexpr (DIM == 3 && VYT == 8) {
            if ((long long)a.n1 * a.n2 * 8 >= (1LL << 31))
                return set_error(FEH_EINVAL, "stencil: one plane of a field must stay below 2 GiB");
            if (unit) hipLaunchKernelGGL((k_stencil<T, 3, ST_TANGENT, true, 8>), grid, block, 0, p.stream, a);
            else hipLaunchKernelGGL((k_stencil<T, 3, ST_TANGENT, false, 8>), grid, block, 0, p.stream, a);
            return hip_check(hipGetLastError(), "tangent launch");
        }
        return set_error(FEH_EINVAL, "bad stencil mode");
    }
    switch (mode) {
        FEH_STENCIL_CASE(ST_APPLY)
        FEH_STENCIL_CASE(ST_CG)
        FEH_STENCIL_CASE(ST_RESID)
        FEH_STENCIL_CASE(ST_DIV)
    default: return set_error(FEH_EINVAL, "bad stencil mode");
    }
#undef FEH_STENCIL_CASE
    return hip_check(hipGetLastError(), "stencil launch");
}

}  // namespace

int stencil_rows(const feh_plan &p) {
    if (p.dim != 3) return 1;
    if (p.tune_stencil_vy == 8 || p.tune_stencil_vy == 16) return p.tune_stencil_vy;
    return 8;
}

int stencil_num_parts(const feh_plan &p) {
    const int n0 = (int)p.n[0];
    const int xc = xchunk(p);
    const int nchunk = (n0 + xc - 1) / xc;
    if (p.dim == 3) {
        const int sy = stencil_rows(p) - 1, sz = 31;
        return nchunk * (int)((p.n[1] + sy - 1) / sy) * (int)((p.n[2] + sz - 1) / sz);
    }
    return nchunk * (int)((p.n[1] + Tile<2, 1>::SZ - 1) / Tile<2, 1>::SZ);
}

int launch_stencil(const feh_plan &p, int mode, const StencilArgs &a) {
    if (p.dim == 2)
        return p.prec == FEH_FP64 ? launch_t<double, 2, 1>(p, mode, a) : launch_t<float, 2, 1>(p, mode, a);
    if (stencil_rows(p) == 16 && mode != ST_TANGENT)
        return p.prec == FEH_FP64 ? launch_t<double, 3, 16>(p, mode, a) : launch_t<float, 3, 16>(p, mode, a);
    return p.prec == FEH_FP64 ? launch_t<double, 3, 8>(p, mode, a) : launch_t<float, 3, 8>(p, mode, a);
}

}  // namespace feh
