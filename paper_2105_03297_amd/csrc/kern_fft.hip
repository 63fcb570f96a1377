// Batched Stockham FFTs staged through LDS, and the per-wavevector
// projection core (B^*B)^-1 fused into the first-axis pass.
//
// The transform pair follows the discrete Fourier transform appendix of the
// paper: forward sum_r f(r) exp(-i k.r) (unnormalised), inverse with 1/N.
// Real fields are transformed along the last (contiguous) axis to the half
// spectrum n_last/2 + 1 (two real samples packed into one complex point and
// untangled with a post-twiddle when n_last is even), then complex-to-complex
// along the other axes.  The spectrum of load case l is stored as
// [n0][(n1)][nh][D], components innermost, so the first-axis pass can read
// all D components of a wavevector in one coalesced segment.
//
// Stockham autosort (each pass reads the previous pass's output layout and
// writes the next, natural order at the end, no bit reversal): pass with
// radix R after earlier radices of product L*, L = L* R, m = n / L:
//   y[q + m (p + L* d)] = sum_c exp(-2 pi i c d / R) w_n^{c p m} x[q + c m + m R p]
// for q < m, p < L*, d < R.
#include <algorithm>
#include <type_traits>

#include "fft_butterflies.hpp"

namespace feh {
namespace {

constexpr int kFftThreads = 256;

// Dynamic LDS holds the twiddle table of the transformed axis (and, in the
// fused first-axis pass, the phase factors of the block's inner wavevector
// indices): staged once per workgroup so the butterflies never wait on global
// memory.
extern __shared__ double feh_dyn_lds[];

// FP64 transforms of general lengths (radix 3..13 and direct passes) are held
// to at most 256 VGPRs, two waves per SIMD; with tiles sized to the pass, two
// workgroups then fit a CU for rows of up to about 1700 points.
// So are the FP32 ones with a prime pass (GEN = 2), whose accumulators else
// take 270 to 340 (FP32, 24 iterations of 6 load cases: 85 x 95 x 115
// 32.9 -> 20.7 ms, 101 x 97 x 89 34.0 -> 21.7, 68^3 8.6 -> 6.9).
template <typename T, int GEN>
constexpr int kGenWaves = (GEN != 0 && sizeof(T) == 8) || GEN == 2 ? 2 : 1;

// LDS one workgroup may hold on gfx950 (160 KiB).  Every launch checks its
// static plus dynamic LDS against it on the host and reports FEH_ENOTSUP
// instead of dispatching a workgroup the hardware cannot allocate.
constexpr size_t kLdsPerWorkgroup = 160 * 1024;

// Streaming global accesses with the nontemporal hint.  The last inverse pass
// uses them for p, u and z: it reads and writes each element of those fields
// once, and nothing reads them again before the next operator pass.  Measured
// per pass, the hint pays only there: on the forward pass (q fresh from the
// stencil) and on the spectrum passes it made the kernels slower.
template <typename T>
__device__ __forceinline__ Cx<T> ldc_nt(const Cx<T> *p) {
    typedef T V __attribute__((ext_vector_type(2)));
    const V v = __builtin_nontemporal_load(reinterpret_cast<const V *>(p));
    return Cx<T>{v.x, v.y};
}
template <typename T>
__device__ __forceinline__ void stc_nt(Cx<T> *p, Cx<T> c) {
    typedef T V __attribute__((ext_vector_type(2)));
    V v;
    v.x = c.x;
    v.y = c.y;
    __builtin_nontemporal_store(v, reinterpret_cast<V *>(p));
}
template <typename T>
__device__ __forceinline__ T ldr_nt(const T *p) { return __builtin_nontemporal_load(p); }
template <typename T>
__device__ __forceinline__ void str_nt(T *p, T v) { __builtin_nontemporal_store(v, p); }

template <typename T>
__device__ __forceinline__ void stage(T *dst, const T *src, int count) {
    for (int i = threadIdx.x; i < count; i += kFftThreads) dst[i] = src[i];
}

// One Stockham pass over nb batches stored interleaved: element j of batch b
// at buf[j * nb + b].  Threads take butterflies batch-fastest so that a
// wavefront reads and writes consecutive LDS words.
template <typename T, int R, int PPT>
__device__ __forceinline__ void stockham_pass(Cx<T> *buf, int nb, const FastDiv &nbd, int n,
                                              const PassInfo &ps, const Cx<T> *tw, int tws, bool inv, int tx) {
    constexpr int NT = kFftThreads;
    constexpr int K = (PPT + R - 1) / R;
    const int nbf = nb * (n / R);
    const int m = (int)ps.m.d;
    const int ostride = m * ps.Lstar * nb;
    Cx<T> y[K][R];
    int obase[K];
    #pragma unroll
    for (int k = 0; k < K; ++k) {
        const int t = tx + k * NT;
        obase[k] = -1;
        if (t < nbf) {
            const int w = (int)nbd.div((uint32_t)t);
            const int b = t - w * nb;
            const int p = (int)ps.m.div((uint32_t)w);
            const int q = w - p * m;
            Cx<T> x[R];
            const int ib = (q + m * R * p) * nb + b;
            #pragma unroll
            for (int c = 0; c < R; ++c) x[c] = buf[ib + c * m * nb];
            if (p != 0) {
                #pragma unroll
                for (int c = 1; c < R; ++c) x[c] = cmul(x[c], twid(tw, tws, c * p * m, inv));
            }
            Dft<T, R>::run(x, inv, tw, tws, n);
            #pragma unroll
            for (int d = 0; d < R; ++d) y[k][d] = x[d];
            obase[k] = (q + m * p) * nb + b;
        }
    }
    __syncthreads();
    #pragma unroll
    for (int k = 0; k < K; ++k) {
        if (obase[k] >= 0) {
            #pragma unroll
            for (int d = 0; d < R; ++d) buf[obase[k] + d * ostride] = y[k][d];
        }
    }
    __syncthreads();
}

// Pass with a prime radix R > 13 (known at run time only) whose tile is too
// narrow for prime_pass (few butterflies of a large prime), each butterfly's
// outputs evaluated directly:
//   y[q + m (p + L* d)] = sum_c w_n^{c m (p + L* d)} x[q + c m + m R p].
// A thread takes B consecutive outputs d0 .. d0 + B - 1 of one butterfly and
// reads each input once: the factor of output d0 + i at term c is
// w_n^{c E0} (w_n^{c n / R})^i with E0 = m (p + L* d0), so per term it reads
// the input and two twiddles from LDS and steps the other B - 1 factors by
// complex multiplication (error growth over at most B - 1 steps).
template <typename T, int PPT>
__device__ __forceinline__ void direct_pass(Cx<T> *buf, int nb, int n, const PassInfo &ps, const Cx<T> *tw, int tws,
                                            bool inv, int tx) {
    constexpr int NT = kFftThreads;
    constexpr int B = 8;
    // work items per thread: items = nb (n / R) ceil(R / B) <= cnt / B + (cnt / R)(B - 1) / B
    // with cnt = nb n <= PPT NT and R >= 17, so at most PPT (17 + B - 1) / (17 B) per thread
    constexpr int KI = (PPT * (17 + B - 1) + 17 * B - 1) / (17 * B);
    const int R = ps.R, m = (int)ps.m.d, Ls = ps.Lstar;
    const int nR = n / R;                       // butterflies per batch (= m L*)
    const int nd = (R + B - 1) / B;             // output blocks per butterfly
    const int items = nb * nR * nd;
    Cx<T> y[KI][B];
    #pragma unroll
    for (int k = 0; k < KI; ++k) {
        const int it = tx + k * NT;
        #pragma unroll
        for (int i = 0; i < B; ++i) y[k][i] = Cx<T>{T(0), T(0)};
        if (it < items) {
            const int b = it % nb;
            const int r1 = it / nb;
            const int db = r1 % nd;
            const int pair = r1 / nd;
            const int q = pair % m;
            const int pp = pair / m;
            const int E0 = m * (pp + Ls * db * B);  // < n
            const int ib = (q + m * R * pp) * nb + b;
            int e0 = 0, es = 0;
            Cx<T> acc[B];
            #pragma unroll
            for (int i = 0; i < B; ++i) acc[i] = Cx<T>{T(0), T(0)};
            for (int c = 0; c < R; ++c) {
                const Cx<T> x = buf[ib + c * m * nb];
                Cx<T> w = twid(tw, tws, e0, inv);
                const Cx<T> st = twid(tw, tws, es, inv);
                #pragma unroll
                for (int i = 0; i < B; ++i) {
                    acc[i] = cadd(acc[i], cmul(x, w));
                    if (i + 1 < B) w = cmul(w, st);
                }
                e0 += E0;
                if (e0 >= n) e0 -= n;
                es += nR;
                if (es >= n) es -= n;
            }
            #pragma unroll
            for (int i = 0; i < B; ++i) y[k][i] = acc[i];
        }
    }
    __syncthreads();
    #pragma unroll
    for (int k = 0; k < KI; ++k) {
        const int it = tx + k * NT;
        if (it < items) {
            const int b = it % nb;
            const int r1 = it / nb;
            const int db = r1 % nd;
            const int pair = r1 / nd;
            const int q = pair % m;
            const int pp = pair / m;
            #pragma unroll
            for (int i = 0; i < B; ++i) {
                const int d = db * B + i;
                if (d < R) buf[(q + m * (pp + Ls * d)) * nb + b] = y[k][i];
            }
        }
    }
    __syncthreads();
}

// Tiles of prime_pass a wavefront may hold: what the accumulators of a
// workgroup's PPT points a thread need, with room for rounding up.
template <int PPT>
constexpr int kPrimeTiles = PPT <= 6 ? 4 : PPT <= 16 ? 8 : 12;
__host__ __device__ inline int prime_tiles(int points, int R) {
    const int rows = ((R - 1) / 2 + 1 + 15) / 16, cols = (2 * (points / R) + 15) / 16;
    return (rows * cols + kFftThreads / 64 - 1) / (kFftThreads / 64);
}

// Pass with a prime radix R > 13 (known at run time only) as a product with
// the matrix cores.  With s_c = x_c + x_{R-c}, d_c = x_c - x_{R-c} (c = 1 ..
// H = (R - 1) / 2, inputs times their Stockham twiddles) the outputs are
//   A_k = x_0 + sum_c s_c cos(2 pi c k / R), B_k = sum_c d_c sin(2 pi c k / R),
//   y_k = A_k -+ i B_k, y_{R-k} = A_k +- i B_k      (k = 0 .. H),
// a quarter of the multiplications of the sum over all c, and two real
// products of a table with the real and imaginary parts of every butterfly
// as columns.  The direct sum (direct_pass, above) spends an LDS read of a
// twiddle for every few multiplications; here a lane reads one table entry
// and two operands for 16 x 16 x 4 x 2 of them.  Measured, FP64 (with the small
// tiles for the first): 151^2 Fourier strain-space solve 22.6 -> 3.3 ms; 1661^2
// FE solve 48.9 -> 19.7 ms.
template <typename T, int PPT>
__device__ __forceinline__ void prime_pass(Cx<T> *buf, int nb, const FastDiv &nbd, int n, const PassInfo &ps,
                                           const Cx<T> *tw, int tws, bool inv, int tx) {
    constexpr int NT = kFftThreads, NW = NT / 64, MT = kPrimeTiles<PPT>;
    using M = Mfma<T>;
    const int R = ps.R, m = (int)ps.m.d, Ls = ps.Lstar, H = (R - 1) / 2;
    const int nR = n / R, bf = nb * nR;         // butterflies
    auto input = [&](int w) {                   // element 0 of butterfly w
        const int r = (int)nbd.div((uint32_t)w), b = w - r * nb;
        const int p = (int)ps.m.div((uint32_t)r), q = r - p * m;
        return (q + m * R * p) * nb + b;
    };
    const int cs = m * nb;                      // between inputs
    // ---- s_c in the place of x_c, d_c in that of x_{R-c}
    for (int i = tx; i < bf * H; i += NT) {
        const int c = 1 + i / bf, w = i - (c - 1) * bf;
        const int r = (int)nbd.div((uint32_t)w);
        const int pm = (int)ps.m.div((uint32_t)r) * m;
        Cx<T> *x0 = buf + input(w);
        Cx<T> x = x0[c * cs], y = x0[(R - c) * cs];
        if (pm != 0) {
            x = cmul(x, twid(tw, tws, c * pm, inv));
            y = cmul(y, twid(tw, tws, (R - c) * pm, inv));
        }
        x0[c * cs] = cadd(x, y);
        x0[(R - c) * cs] = csub(x, y);
    }
    __syncthreads();
    // ---- tiles of 16 outputs k by 16 columns (8 butterflies, real and imaginary)
    const int lane = tx & 63, wv = tx >> 6, li = lane & 15, lg = lane >> 4;
    const int KT = (H + 1 + 15) / 16, CT = (2 * bf + 15) / 16;
    typename M::Acc A[MT], B[MT];
    const T *re = reinterpret_cast<const T *>(buf);
    #pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int t = wv + NW * i;
        if (t < KT * CT) {                      // the same for the whole wavefront
            const int ct = t / KT, kt = t - ct * KT;
            const int col = ct * 16 + li, w = col >> 1;
            const bool on = w < bf;
            const T *x0 = re + 2 * input(on ? w : 0) + (col & 1);
            const int k = min(kt * 16 + li, H);
            const T first = on ? x0[0] : T(0);
            typename M::Acc a = {first, first, first, first}, b = {T(0), T(0), T(0), T(0)};
            int c = 1 + lg;
            int e = (c * k) % R;
            const int step = (4 * k) % R;
            for (int c0 = 1; c0 <= H; c0 += 4) {
                const Cx<T> wt = tw[e * nR * tws];  // cos, -sin
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
    T *out = reinterpret_cast<T *>(buf);
    const int os = m * Ls * nb;                 // between outputs
    #pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int t = wv + NW * i;
        if (t < KT * CT) {
            const int ct = t / KT, kt = t - ct * KT;
            const int col = ct * 16 + li, w = col >> 1;
            const int r1 = (int)nbd.div((uint32_t)w), b1 = w - r1 * nb;
            const int p = (int)ps.m.div((uint32_t)r1), q = r1 - p * m;
            T *y0 = out + 2 * ((q + m * p) * nb + b1) + (col & 1);
            #pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k = kt * 16 + M::row(lane, r);
                // -i B = (B_im, -B_re), the other part being the neighbouring
                // column's; + i B for the inverse
                const T bx = __shfl_xor(B[i][r], 1);
                const T ib = ((col & 1) != 0) == inv ? bx : -bx;
                if (w < bf && k <= H) {
                    y0[2 * k * os] = A[i][r] + ib;
                    if (k > 0) y0[2 * (R - k) * os] = A[i][r] - ib;
                }
            }
        }
    }
    __syncthreads();
}

// Passes that an instantiation holds, so that a length does not pay the
// registers of passes it has none of: GEN = 0 the radices of power-of-two
// lengths (2, 4, 8), 1 also 3 to 13, 2 also the prime passes (the matrix-core
// accumulators of prime_pass in the kernels of lengths without a prime above
// 13 took a solve on 90 x 77 x 105 in FP32 from 11.1 to 16.1 ms).
template <typename T, int PPT, int GEN>
__device__ __forceinline__ void lds_fft(Cx<T> *buf, int nb, const FastDiv &nbd, const AxisFFT &ax,
                                        const Cx<T> *tw, int tws, bool inv, int tx = threadIdx.x) {
    for (int s = 0; s < ax.npass; ++s) {
        const PassInfo &ps = ax.pass[s];
        switch (ps.R) {
        case 2: stockham_pass<T, 2, PPT>(buf, nb, nbd, ax.n, ps, tw, tws, inv, tx); break;
        case 4: stockham_pass<T, 4, PPT>(buf, nb, nbd, ax.n, ps, tw, tws, inv, tx); break;
        case 8: stockham_pass<T, 8, PPT>(buf, nb, nbd, ax.n, ps, tw, tws, inv, tx); break;
        default:
            if constexpr (GEN != 0) {
                switch (ps.R) {
                case 3: stockham_pass<T, 3, PPT>(buf, nb, nbd, ax.n, ps, tw, tws, inv, tx); break;
                case 5: stockham_pass<T, 5, PPT>(buf, nb, nbd, ax.n, ps, tw, tws, inv, tx); break;
                case 7: stockham_pass<T, 7, PPT>(buf, nb, nbd, ax.n, ps, tw, tws, inv, tx); break;
                case 11: stockham_pass<T, 11, PPT>(buf, nb, nbd, ax.n, ps, tw, tws, inv, tx); break;
                case 13: stockham_pass<T, 13, PPT>(buf, nb, nbd, ax.n, ps, tw, tws, inv, tx); break;
                default:
                    if constexpr (GEN == 2) {
                        if (prime_tiles(nb * ax.n, ps.R) <= kPrimeTiles<PPT>)
                            prime_pass<T, PPT>(buf, nb, nbd, ax.n, ps, tw, tws, inv, tx);
                        else direct_pass<T, PPT>(buf, nb, ax.n, ps, tw, tws, inv, tx);
                    }
                    break;
                }
            }
            break;
        }
    }
}

template <typename T>
struct FK {
    const T *r;
    const T *q;
    T *r_out;
    Cx<T> *spec;
    const Cx<T> *spec_in;     // middle pass: read from here, write spec (null: in place)
    T *z;
    T *p_upd;                 // fused CG update in the last inverse pass
    void *u_upd;              // T, or double in the accumulating variant (U of the kernels)
    double *partial;
    const LcState *st;
    const Cx<T> *tw;          // twiddles of the transformed axis (full length)
    int tws;                  // table stride (2 for the packed last axis)
    const Cx<T> *tw_last;     // last-axis table (post-twiddle of the packed transform)
    const double *om[3];      // e^{2 pi i m / n_a}, interleaved complex
    const double *aa[3];      // (e^{2 pi i m / n_a} - 1) / h_a
    AxisFFT ax;
    FastDiv nbd;              // batches per block
    FastDiv d_nc;             // packed length / FFT length
    FastDiv d_D;              // components
    FastDiv d_nhD;            // nh * D
    FastDiv d_PB;             // pencils per block
    FastDiv d_nh;
    int dim, D, L;
    int n0, n1, nlast, nh;
    long long N, rows, inner_total;
    int RR, PB, nblk, total;
    int lbuf;                 // entries of the LDS tile (last and middle passes): the
                              // dynamic LDS holds the tile, then the twiddle table
    int part_stride;
    int last_even;
    int use_axpy;             // selects the AXPY instantiation on the host
    double out_scale, invN, chalf;  // chalf = element volume / 2
    float near0;              // FP32 plans: sum_a |aa_a|^2 below which M^-1 is formed in FP64
    float hmax_f, post_f;     // FP32 plans: h_max and h_max^2 / chalf (scale-free FP32 inverse)
    int metric;               // feh_plan::metric, and for 1 + kind the point weight and the smallest symbol
    double metric_w, metric_tiny;
    T *minv;                  // (B^*B)^-1 table [block][component][slot] (first-axis pass)
    int minv_q;               // 0: slots in order; Q: interleaved for Q-wide loads (see minv_pos)
};

// Position of wavevector slot e in a block's table row.  With q > 0 the
// slots of each run of 64 q are interleaved so that lane l's q-wide vector
// load holds slots l, l + 64, .., l + 64 (q - 1) of the run: a wavefront then
// takes 64 consecutive slots per vector element (consecutive LDS words in the
// first-axis pass) while each lane still loads 16 contiguous bytes.
__host__ __device__ inline int minv_pos(int e, int q) {
    if (q == 0) return e;
    const int run = 64 * q;
    return (e / run) * run + (e % 64) * q + (e % run) / 64;
}

// ---------------------------------------------------------------------------
// Transforms with the shape fixed at compile time: power-of-two length N in
// the plan's default radix order (8 while it divides, then 4 or 2), DS
// sub-problems of NB batches each (NB a power of two), element j of batch b
// of sub-problem s at buf[(s N + j) NB + b].  Every thread index splits into
// (sub-problem, butterfly, batch) by shifts and masks, the LDS offsets of a
// butterfly are compile-time strides and the passes unroll, so the index
// arithmetic that the run-time passes spend in integer multiplies and
// divisions (quarter-rate on this chip) and in bounds branches disappears.
// The butterflies and twiddles are those of stockham_pass, in the same
// order, so the results are the same numbers.
// ---------------------------------------------------------------------------
constexpr int ct_radix_at(int n, int s) {
    int m = n, r = 1;
    for (int i = 0; i <= s; ++i) {
        r = (m % 8 == 0) ? 8 : (m % 4 == 0) ? 4 : 2;
        m /= r;
    }
    return r;
}
constexpr int ct_npass(int n) {
    int k = 0;
    for (int m = n; m > 1; ++k) m /= (m % 8 == 0) ? 8 : (m % 4 == 0) ? 4 : 2;
    return k;
}
constexpr int ct_lstar(int n, int s) {
    int L = 1;
    for (int i = 0; i < s; ++i) L *= ct_radix_at(n, i);
    return L;
}
constexpr int ct_log2(int x) {
    int l = 0;
    while ((1 << l) < x) ++l;
    return l;
}

// Does the run-time schedule of an axis equal the compile-time one of length n?
__host__ inline bool ct_schedule_matches(const AxisFFT &ax, int n) {
    if (ax.n != n || ax.npass != ct_npass(n)) return false;
    for (int s = 0; s < ax.npass; ++s)
        if (ax.pass[s].R != ct_radix_at(n, s)) return false;
    return true;
}

// floor(x / DV) for 0 <= x < RANGE: a shift for powers of two, otherwise
// one full-rate 24-bit multiply by a magic constant and a shift, the
// constant searched and checked over the whole range at compile time.
template <int DV, int RANGE>
struct CtDiv {
    static constexpr bool pow2 = (DV & (DV - 1)) == 0;
    static constexpr bool exact(int sh, unsigned long long m) {
        for (int x = 0; x < RANGE; ++x)
            if ((unsigned long long)x * m >> sh != (unsigned long long)(x / DV)) return false;
        return true;
    }
    static constexpr int find() {
        if (pow2) return ct_log2(DV);
        for (int sh = 0; sh < 32; ++sh) {
            const unsigned long long m = (1ull << sh) / DV + 1;
            if (m < (1ull << 24) && (unsigned long long)(RANGE - 1) * m < (1ull << 32) && exact(sh, m)) return sh;
        }
        return -1;
    }
    static constexpr int SH = find();
    static constexpr unsigned MG = pow2 ? 1u : (unsigned)((1ull << (SH < 0 ? 0 : SH)) / DV + 1);
    static_assert(SH >= 0, "no 24-bit magic divisor for this range");
    static __device__ __forceinline__ int div(int x) {
        if constexpr (pow2) return x >> SH;
        else return (int)(__umul24((unsigned)x, MG) >> SH);
    }
};

// Element j of batch b of sub-problem s sits at buf[(s N + j) NBS + b]; a
// row stride NBS > NB (odd) spreads the lanes of a stride-NBS access over the
// LDS banks.
template <typename T, int N, int NB, int DS, int S, bool INV, int TWS = 1, int NBS = NB>
__device__ __forceinline__ void ct_pass(Cx<T> *buf, const Cx<T> *tw) {
    constexpr int NT = kFftThreads;
    constexpr int R = ct_radix_at(N, S), LS = ct_lstar(N, S);
    constexpr int M = N / (LS * R), BF = N / R;
    constexpr int ITEMS = DS * BF * NB;
    constexpr int K = (ITEMS + NT - 1) / NT;
    constexpr bool EXACT = ITEMS % NT == 0;  // else the last round has idle threads
    constexpr int LBF = ct_log2(BF), LM = ct_log2(M);
    Cx<T> y[K][R];
    int ob[K];
    #pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i0 = threadIdx.x + k * NT;
        const bool on = EXACT || i0 < ITEMS;
        const int i = on ? i0 : 0;
        const int wq = CtDiv<NB, ITEMS>::div(i);  // butterfly index over all sub-problems
        const int b = i - wq * NB;
        const int w = wq & (BF - 1);
        const int sb = (wq >> LBF) * (N * NBS) + b;
        const int p = w >> LM, q = w & (M - 1);
        const int ib = sb + (q + ((p * R) << LM)) * NBS;
        Cx<T> x[R];
        #pragma unroll
        for (int c = 0; c < R; ++c) x[c] = buf[ib + c * M * NBS];
        if constexpr (LS > 1) {
            // butterflies with p = 0 multiply by the twiddle 1 (exact), so
            // the lanes of a wave take no divergent branch
            const int pm = p << LM;
            #pragma unroll
            for (int c = 1; c < R; ++c) x[c] = cmul(x[c], twid(tw, TWS, c * pm, INV));
        }
        Dft<T, R>::run(x, INV, tw, 1, N);
        #pragma unroll
        for (int d = 0; d < R; ++d) y[k][d] = x[d];
        ob[k] = sb + (q + (p << LM)) * NBS;
        if (!on) ob[k] = -1;
    }
    __syncthreads();
    #pragma unroll
    for (int k = 0; k < K; ++k) {
        if (EXACT || ob[k] >= 0) {
            #pragma unroll
            for (int d = 0; d < R; ++d) buf[ob[k] + d * (M * LS * NBS)] = y[k][d];
        }
    }
    __syncthreads();
}

// Passes S .. E - 1 (E = all of them by default).
template <typename T, int N, int NB, int DS, int S, bool INV, int TWS, int NBS, int E = ct_npass(N)>
__device__ __forceinline__ void ct_passes(Cx<T> *buf, const Cx<T> *tw) {
    if constexpr (S < E) {
        ct_pass<T, N, NB, DS, S, INV, TWS, NBS>(buf, tw);
        ct_passes<T, N, NB, DS, S + 1, INV, TWS, NBS, E>(buf, tw);
    }
}

// The whole transform (the buffer already staged and synchronised); the
// twiddle table holds e^{-2 pi i j / (N TWS)} at j (TWS = 2: the table of the
// unpacked length of a packed real transform).
template <typename T, int N, int NB, int DS, bool INV, int TWS = 1, int NBS = NB>
__device__ __forceinline__ void ct_fft(Cx<T> *buf, const Cx<T> *tw) {
    ct_passes<T, N, NB, DS, 0, INV, TWS, NBS>(buf, tw);
}

// Pencils of a compile-time pass per workgroup: N NB points, 16 per thread in
// FP32 (32 KiB of LDS) and 8 in FP64, so that four (FP32) or two (FP64)
// workgroups share a CU.
template <typename T, int N>
constexpr int ct_batches() { return (sizeof(T) == 4 ? 16 : 8) * kFftThreads / N; }

// ---------------------------------------------------------------------------
// last axis, real -> half spectrum (AXPY: fused r -= alpha q, r written back)
//
// Global memory is touched in two phases per kernel: every load of a thread
// is issued before the first use (indices of slots past the end are clamped
// into the block so the loads stay in bounds; their values are discarded),
// then every store; r and r_out may be the same buffer.
// ---------------------------------------------------------------------------
template <typename T, int PPT, int GEN, bool AXPY>
__global__ __launch_bounds__(kFftThreads) __attribute__((amdgpu_waves_per_eu(kGenWaves<T, GEN>))) void k_last_fwd(FK<T> a) {
    constexpr int NT = kFftThreads;
    __shared__ Cx<T> sbuf[GEN ? 1 : PPT * NT];
    Cx<T> *buf = GEN ? reinterpret_cast<Cx<T> *>(feh_dyn_lds) : sbuf;
    int t = xcd_remap(blockIdx.x, a.total);
    const int lc = t / a.nblk;
    const int blk = t - lc * a.nblk;
    T alpha = T(0);
    if (a.st) {
        if (!a.st[lc].active) return;
        if (AXPY) alpha = T(a.st[lc].alpha);
    }
    const int D = a.D;
    const int nb = D * a.RR;
    const long long s0 = (long long)blk * a.RR;
    const int nrows = (int)min((long long)a.RR, a.rows - s0);
    const int nc = a.ax.n;
    const int cnt = nb * nc;
    const long long N = a.N;
    const int even = a.last_even;
    Cx<T> *twl = GEN ? buf + a.lbuf : reinterpret_cast<Cx<T> *>(feh_dyn_lds);
    stage(twl, a.tw_last, a.nlast);
    const long long lbase = (long long)lc * D * N + s0 * a.nlast;
    // AXPY keeps two loads per slot in flight: 8 slots per round
    constexpr int CH = AXPY && PPT > 8 ? 8 : PPT;
    #pragma unroll
    for (int h = 0; h < PPT; h += CH) {
        Cx<T> v[CH];
        Cx<T> w[AXPY ? CH : 1];
        #pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int e0 = threadIdx.x + (h + k) * NT;
            const int e = e0 < cnt ? e0 : 0;
            const int b = (int)a.d_nc.div((uint32_t)e);
            const int j = e - b * nc;
            const int sl0 = (int)a.d_D.div((uint32_t)b);
            const int c = b - sl0 * D;
            const int sl = sl0 < nrows ? sl0 : nrows - 1;
            // element offset of the packed pair (even) or of the sample (odd)
            const long long off = lbase + (long long)c * N + (long long)sl * a.nlast + (even ? 2 * j : j);
            if (even) {
                v[k] = *reinterpret_cast<const Cx<T> *>(a.r + off);
                if (AXPY) w[k] = *reinterpret_cast<const Cx<T> *>(a.q + off);
            } else {
                v[k] = Cx<T>{a.r[off], T(0)};
                if (AXPY) w[k] = Cx<T>{a.q[off], T(0)};
            }
        }
        #pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int e0 = threadIdx.x + (h + k) * NT;
            const int e = e0 < cnt ? e0 : 0;
            const int b = (int)a.d_nc.div((uint32_t)e);
            const int j = e - b * nc;
            const int sl = (int)a.d_D.div((uint32_t)b);
            const int c = b - sl * D;
            const bool ok = e0 < cnt && sl < nrows;
            if (AXPY) {
                v[k].x -= alpha * w[k].x;
                v[k].y -= alpha * w[k].y;
                if (ok) {
                    const long long off = lbase + (long long)c * N + (long long)sl * a.nlast + (even ? 2 * j : j);
                    if (even) *reinterpret_cast<Cx<T> *>(a.r_out + off) = v[k];
                    else a.r_out[off] = v[k].x;
                }
            }
            if (!ok) v[k] = Cx<T>{T(0), T(0)};
            if (e0 < cnt) buf[j * nb + b] = v[k];
        }
    }
    __syncthreads();
    lds_fft<T, PPT, GEN>(buf, nb, a.nbd, a.ax, twl, a.tws, false);
    // untangle the packed transform and store the half spectrum, components
    // fastest; the count nrows * nh * D exceeds PPT * NT by at most nb
    const int nh = a.nh;
    const int ocnt = nrows * nh * D;
    Cx<T> X[PPT + 1];
    #pragma unroll
    for (int k = 0; k < PPT + 1; ++k) {
        const int e0 = threadIdx.x + k * NT;
        const int e = e0 < ocnt ? e0 : 0;
        const int kk = (int)a.d_D.div((uint32_t)e);
        const int c = e - kk * D;
        const int sl = (int)a.d_nh.div((uint32_t)kk);
        const int kx = kk - sl * nh;
        const int b = sl * D + c;
        if (even) {
            const int ka = (kx == nc) ? 0 : kx;
            const int kb = (kx == 0) ? 0 : nc - kx;
            const Cx<T> Zk = buf[ka * nb + b], Zm = cconj(buf[kb * nb + b]);
            const Cx<T> A = {T(0.5) * (Zk.x + Zm.x), T(0.5) * (Zk.y + Zm.y)};
            const Cx<T> dZ = csub(Zk, Zm);
            const Cx<T> B = {T(0.5) * dZ.y, -T(0.5) * dZ.x};  // -i/2 (Zk - conj Z(nc-k))
            X[k] = cadd(A, cmul(twl[kx], B));
        } else {
            X[k] = buf[kx * nb + b];
        }
    }
    Cx<T> *dst = a.spec + ((long long)lc * a.rows + s0) * (long long)nh * D;
    #pragma unroll
    for (int k = 0; k < PPT + 1; ++k) {
        const int e0 = threadIdx.x + k * NT;
        if (e0 < ocnt) dst[e0] = X[k];
    }
}

// ---------------------------------------------------------------------------
// last axis, half spectrum -> real (times out_scale).  UPD: the real result z
// is not stored; instead the CG update u += alpha_pend p, p = z + beta p is
// applied in place (one pass over p and u while z is in registers).  U: the
// type u is kept in (T, or double in an FP32 plan whose caller differentiates
// u and must not lose the digits that its rounding to float would take).
// ---------------------------------------------------------------------------
template <typename T, int PPT, int GEN, bool UPD, typename U = T>
__global__ __launch_bounds__(kFftThreads) __attribute__((amdgpu_waves_per_eu(kGenWaves<T, GEN>))) void k_last_inv(FK<T> a) {
    constexpr int NT = kFftThreads;
    __shared__ Cx<T> sbuf[GEN ? 1 : PPT * NT];
    Cx<T> *buf = GEN ? reinterpret_cast<Cx<T> *>(feh_dyn_lds) : sbuf;
    int t = xcd_remap(blockIdx.x, a.total);
    const int lc = t / a.nblk;
    const int blk = t - lc * a.nblk;
    if (a.st && !a.st[lc].active) return;
    const int D = a.D;
    const int nb = D * a.RR;
    const long long s0 = (long long)blk * a.RR;
    const int nrows = (int)min((long long)a.RR, a.rows - s0);
    const int nc = a.ax.n;
    const int nh = a.nh;
    const int cnt = nb * nc;
    const long long N = a.N;
    const int even = a.last_even;
    Cx<T> *twl = GEN ? buf + a.lbuf : reinterpret_cast<Cx<T> *>(feh_dyn_lds);
    stage(twl, a.tw_last, a.nlast);
    __syncthreads();
    // gather e -> (sl, k, c), components fastest (coalesced spectrum reads);
    // the packed input Z(k) needs X(k) and X(nc - k)
    const Cx<T> *src = a.spec + ((long long)lc * a.rows + s0) * (long long)nh * D;
    constexpr int CH = PPT / 2;
    #pragma unroll
    for (int h = 0; h < PPT; h += CH) {
        Cx<T> Xa[CH], Xb[CH];
        #pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int e0 = threadIdx.x + (h + k) * NT;
            const int e = e0 < cnt ? e0 : 0;
            const int kk = (int)a.d_D.div((uint32_t)e);
            const int c = e - kk * D;
            const int sl0 = (int)a.d_nc.div((uint32_t)kk);
            const int kx = kk - sl0 * nc;
            const int sl = sl0 < nrows ? sl0 : nrows - 1;
            const Cx<T> *row = src + (long long)sl * nh * D + c;
            if (even) {
                Xa[k] = row[(long long)kx * D];
                Xb[k] = row[(long long)(nc - kx) * D];
            } else {
                Xa[k] = row[(long long)(kx < nh ? kx : a.nlast - kx) * D];
            }
        }
        #pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int e0 = threadIdx.x + (h + k) * NT;
            const int e = e0 < cnt ? e0 : 0;
            const int kk = (int)a.d_D.div((uint32_t)e);
            const int c = e - kk * D;
            const int sl = (int)a.d_nc.div((uint32_t)kk);
            const int kx = kk - sl * nc;
            // the DC and Nyquist samples of a real signal's spectrum are real:
            // their imaginary parts (rounding residue) are dropped
            if (kx == 0) {
                Xa[k].y = T(0);
                Xb[k].y = T(0);
            }
            Cx<T> Z;
            if (even) {
                const Cx<T> Xm = cconj(Xb[k]);
                const Cx<T> A = cadd(Xa[k], Xm);
                const Cx<T> B = cmulc(csub(Xa[k], Xm), twl[kx]);  // exp(+2 pi i k / n) (Xk - conj X(nc-k))
                Z = cadd(A, mul_pi(B));
            } else {
                Z = kx < nh ? Xa[k] : cconj(Xa[k]);
            }
            if (sl >= nrows) Z = Cx<T>{T(0), T(0)};
            if (e0 < cnt) buf[kx * nb + sl * D + c] = Z;
        }
    }
    __syncthreads();
    lds_fft<T, PPT, GEN>(buf, nb, a.nbd, a.ax, twl, a.tws, true);
    const T sc = T(a.out_scale);
    Cx<T> y[PPT];
    #pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int e0 = threadIdx.x + k * NT;
        const int e = e0 < cnt ? e0 : 0;
        const int b = (int)a.d_nc.div((uint32_t)e);
        const int j = e - b * nc;
        y[k] = buf[j * nb + b];
    }
    const long long lbase = (long long)lc * D * N + s0 * a.nlast;
    if constexpr (UPD) {
        const T beta = T(a.st[lc].beta);
        const U ap = U(a.st[lc].alpha_pend);
        U *uu = static_cast<U *>(a.u_upd);
        constexpr int CH = PPT > 8 ? 8 : PPT;  // slots per round: two loads each in flight
        #pragma unroll
        for (int h = 0; h < PPT; h += CH) {
            Cx<T> pv[CH];
            Cx<U> uv[CH];
            #pragma unroll
            for (int k = 0; k < CH; ++k) {
                const int e0 = threadIdx.x + (h + k) * NT;
                const int e = e0 < cnt ? e0 : 0;
                const int b = (int)a.d_nc.div((uint32_t)e);
                const int j = e - b * nc;
                const int sl0 = (int)a.d_D.div((uint32_t)b);
                const int c = b - sl0 * D;
                const int sl = sl0 < nrows ? sl0 : nrows - 1;
                const long long o = lbase + (long long)c * N + (long long)sl * a.nlast + (even ? 2 * j : j);
                if (even) {
                    pv[k] = ldc_nt(reinterpret_cast<const Cx<T> *>(a.p_upd + o));
                    uv[k] = ldc_nt(reinterpret_cast<const Cx<U> *>(uu + o));
                } else {
                    pv[k] = Cx<T>{ldr_nt(a.p_upd + o), T(0)};
                    uv[k] = Cx<U>{ldr_nt(uu + o), U(0)};
                }
            }
            #pragma unroll
            for (int k = 0; k < CH; ++k) {
                const int e0 = threadIdx.x + (h + k) * NT;
                const int b = (int)a.d_nc.div((uint32_t)e0);
                const int j = e0 - b * nc;
                const int sl = (int)a.d_D.div((uint32_t)b);
                const int c = b - sl * D;
                if (e0 < cnt && sl < nrows) {
                    const long long o = lbase + (long long)c * N + (long long)sl * a.nlast + (even ? 2 * j : j);
                    const Cx<T> z = {y[h + k].x * sc, y[h + k].y * sc};
                    const Cx<U> un = {uv[k].x + ap * U(pv[k].x), uv[k].y + ap * U(pv[k].y)};
                    const Cx<T> pn = {z.x + beta * pv[k].x, z.y + beta * pv[k].y};
                    if (even) {
                        stc_nt(reinterpret_cast<Cx<U> *>(uu + o), un);
                        stc_nt(reinterpret_cast<Cx<T> *>(a.p_upd + o), pn);
                    } else {
                        str_nt(uu + o, un.x);
                        str_nt(a.p_upd + o, pn.x);
                    }
                }
            }
        }
    } else {
        #pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const int e0 = threadIdx.x + k * NT;
            const int b = (int)a.d_nc.div((uint32_t)e0);
            const int j = e0 - b * nc;
            const int sl = (int)a.d_D.div((uint32_t)b);
            const int c = b - sl * D;
            if (e0 < cnt && sl < nrows) {
                const long long o = lbase + (long long)c * N + (long long)sl * a.nlast;
                if (even) stc_nt(reinterpret_cast<Cx<T> *>(a.z + o) + j, Cx<T>{y[k].x * sc, y[k].y * sc});
                else str_nt(a.z + o + j, y[k].x * sc);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Last-axis passes with the compile-time transform: even length NL (packed
// into NC = NL / 2 complex points) in the default radix order, RR rows of D
// components per workgroup (24 points per thread in FP32), the LDS tile and
// the global layouts of k_last_fwd / k_last_inv (batch b = row D + component,
// element j at buf[j NBS + b], NBS = ct_last_stride).  Same arithmetic in the
// same order.
// ---------------------------------------------------------------------------
template <int NL, int D>
constexpr int ct_last_rows() { return 24 * kFftThreads / (NL / 2 * D); }
// LDS row stride of the tile: one past the D RR batches (odd, so that the
// transposing accesses, consecutive lanes one row apart, hit distinct banks)
// when three workgroups still fit a CU's LDS with it, else D RR
template <int NL, int D>
constexpr int ct_last_stride() {
    constexpr int NB = D * ct_last_rows<NL, D>();
    return (NB + 1) * (NL / 2) * 8 + NL * 8 <= 160 * 1024 / 3 ? NB + 1 : NB;
}

// Byte offset of packed pair j of row sl (of the block) and component c in
// the load case's real SoA field [D][N].
template <typename T, int NL, int D>
__device__ __forceinline__ unsigned last_pair_offset(int c, int sl, int j, unsigned N32, unsigned row0) {
    // c N: N is a multiple of NL >= 128, so one 24-bit multiply of N / 128
    static_assert(NL % 128 == 0, "component stride from N / 128");
    const unsigned cb = __umul24((unsigned)c, N32 >> 7) << 7;
    return (cb + row0 + (unsigned)(sl * NL + 2 * j)) * (unsigned)sizeof(T);
}

// MODE 0: r -> half spectrum; MODE 1 (AXPY): r -= alpha q, r written back, its
// half spectrum written; MODE 2 (RSPEC): the half spectrum of q, and the
// residual kept as a half spectrum updated in place, spec -= alpha q^.
template <typename T, int NL, int D, int MODE, bool FULL>
__device__ __forceinline__ void last_fwd_ct_body(const FK<T> &a, int lc, long long s0, int nrows, T alpha,
                                                 Cx<T> *buf, const Cx<T> *twl) {
    constexpr int NT = kFftThreads, NC = NL / 2, NH = NC + 1;
    constexpr int RR = ct_last_rows<NL, D>(), NB = D * RR, NBS = ct_last_stride<NL, D>();
    constexpr int CNT = NB * NC, PPT = CNT / NT;
    constexpr int OCNT = RR * NH * D;                  // half-spectrum values of the block
    constexpr int KO = (OCNT + NT - 1) / NT;
    constexpr int LNC = ct_log2(NC);
    const long long lbase = (long long)lc * D * a.N;
    constexpr bool AXPY = MODE == 1;
    const T *rl = MODE == 2 ? a.q + lbase : a.r + lbase;  // the transformed field
    const T *ql = AXPY ? a.q + lbase : nullptr;
    T *rol = AXPY ? a.r_out + lbase : nullptr;
    const unsigned N32 = (unsigned)a.N, row0 = (unsigned)(s0 * NL);
    // slot e -> batch b = e / NC (row sl = b / D, component c), packed pair j
    constexpr int CH = AXPY ? 8 : PPT;
    #pragma unroll
    for (int h = 0; h < PPT; h += CH) {
        Cx<T> v[CH];
        Cx<T> w[AXPY ? CH : 1];
        #pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int e = threadIdx.x + (h + k) * NT;
            const int b = e >> LNC, j = e & (NC - 1);
            const int sl0 = CtDiv<D, NB>::div(b), c = b - sl0 * D;
            const int sl = (FULL || sl0 < nrows) ? sl0 : nrows - 1;
            const unsigned off = last_pair_offset<T, NL, D>(c, sl, j, N32, row0);
            v[k] = *at_byte(reinterpret_cast<const Cx<T> *>(rl), off);
            if (AXPY) w[k] = *at_byte(reinterpret_cast<const Cx<T> *>(ql), off);
        }
        #pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int e = threadIdx.x + (h + k) * NT;
            const int b = e >> LNC, j = e & (NC - 1);
            const int sl = CtDiv<D, NB>::div(b), c = b - sl * D;
            const bool ok = FULL || sl < nrows;
            if (AXPY) {
                v[k].x -= alpha * w[k].x;
                v[k].y -= alpha * w[k].y;
                if (ok) *at_byte(reinterpret_cast<Cx<T> *>(rol), last_pair_offset<T, NL, D>(c, sl, j, N32, row0)) = v[k];
            }
            buf[j * NBS + b] = ok ? v[k] : Cx<T>{T(0), T(0)};
        }
    }
    __syncthreads();
    ct_fft<T, NC, NB, 1, false, 2, NBS>(buf, twl);
    // untangle the packed transform; half spectrum out, components fastest
    Cx<T> X[KO];
    #pragma unroll
    for (int k = 0; k < KO; ++k) {
        const int e0 = threadIdx.x + k * NT;
        const int e = (OCNT % NT == 0 || e0 < OCNT) ? e0 : 0;
        const int kk = CtDiv<D, OCNT>::div(e);
        const int c = e - kk * D;
        const int sl = CtDiv<NH, OCNT / D>::div(kk);
        const int kx = kk - sl * NH;
        const int b = sl * D + c;
        const int ka = (kx == NC) ? 0 : kx;
        const int kb = (kx == 0) ? 0 : NC - kx;
        const Cx<T> Zk = buf[ka * NBS + b], Zm = cconj(buf[kb * NBS + b]);
        const Cx<T> A = {T(0.5) * (Zk.x + Zm.x), T(0.5) * (Zk.y + Zm.y)};
        const Cx<T> dZ = csub(Zk, Zm);
        const Cx<T> B = {T(0.5) * dZ.y, -T(0.5) * dZ.x};  // -i/2 (Zk - conj Z(nc-k))
        X[k] = cadd(A, cmul(twl[kx], B));
    }
    Cx<T> *dst = a.spec + ((long long)lc * a.rows + s0) * (long long)NH * D;
    const int ocnt = FULL ? OCNT : nrows * NH * D;
    if constexpr (MODE == 2) {
        // every load before the first store
        Cx<T> R[KO];
        #pragma unroll
        for (int k = 0; k < KO; ++k) {
            const int e0 = threadIdx.x + k * NT;
            const int e = ((FULL && (OCNT % NT == 0 || k + 1 < KO)) || e0 < ocnt) ? e0 : 0;
            R[k] = *at_byte(dst, (unsigned)e * (unsigned)sizeof(Cx<T>));
        }
        #pragma unroll
        for (int k = 0; k < KO; ++k) {
            const int e0 = threadIdx.x + k * NT;
            if ((FULL && (OCNT % NT == 0 || k + 1 < KO)) || e0 < ocnt)
                *at_byte(dst, (unsigned)e0 * (unsigned)sizeof(Cx<T>)) =
                    Cx<T>{R[k].x - alpha * X[k].x, R[k].y - alpha * X[k].y};
        }
    } else {
        #pragma unroll
        for (int k = 0; k < KO; ++k) {
            const int e0 = threadIdx.x + k * NT;
            if ((FULL && (OCNT % NT == 0 || k + 1 < KO)) || e0 < ocnt) *at_byte(dst, (unsigned)e0 * (unsigned)sizeof(Cx<T>)) = X[k];
        }
    }
}

template <typename T, int NL, int D, int MODE>
__global__ __launch_bounds__(kFftThreads) void k_last_fwd_ct(FK<T> a) {
    constexpr int NT = kFftThreads, NC = NL / 2;
    constexpr int RR = ct_last_rows<NL, D>(), NB = D * RR;
    static_assert((NB * NC) % NT == 0, "whole slots per thread");
    __shared__ Cx<T> buf[ct_last_stride<NL, D>() * NC];
    __shared__ Cx<T> twl[NL];
    const int t = xcd_remap(blockIdx.x, a.total);
    const int lc = t / a.nblk;
    const int blk = t - lc * a.nblk;
    T alpha = T(0);
    if (a.st) {
        if (!a.st[lc].active) return;
        if (MODE != 0) alpha = T(a.st[lc].alpha);
    }
    const long long s0 = (long long)blk * RR;
    const int nrows = (int)min((long long)RR, a.rows - s0);
    for (int i = threadIdx.x; i < NL; i += NT) twl[i] = a.tw_last[i];
    if (nrows == RR) last_fwd_ct_body<T, NL, D, MODE, true>(a, lc, s0, nrows, alpha, buf, twl);
    else last_fwd_ct_body<T, NL, D, MODE, false>(a, lc, s0, nrows, alpha, buf, twl);
}

template <typename T, int NL, int D, bool UPD, bool FULL, typename U>
__device__ __forceinline__ void last_inv_ct_body(const FK<T> &a, int lc, long long s0, int nrows, Cx<T> *buf,
                                                 const Cx<T> *twl) {
    constexpr int NT = kFftThreads, NC = NL / 2, NH = NC + 1;
    constexpr int RR = ct_last_rows<NL, D>(), NB = D * RR, NBS = ct_last_stride<NL, D>();
    constexpr int CNT = NB * NC, PPT = CNT / NT;
    constexpr int LNC = ct_log2(NC);
    // gather e -> (row sl, k, component c), components fastest; the packed
    // input Z(k) needs X(k) and X(nc - k)
    const Cx<T> *src = a.spec + ((long long)lc * a.rows + s0) * (long long)NH * D;
    constexpr int CH = PPT / 2;
    #pragma unroll
    for (int h = 0; h < PPT; h += CH) {
        Cx<T> Xa[CH], Xb[CH];
        #pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int e = threadIdx.x + (h + k) * NT;
            const int kk = CtDiv<D, CNT>::div(e);
            const int c = e - kk * D;
            const int sl0 = kk >> LNC, kx = kk & (NC - 1);
            const int sl = (FULL || sl0 < nrows) ? sl0 : nrows - 1;
            const unsigned row = (unsigned)(sl * (NH * D) + c);
            Xa[k] = *at_byte(src, (row + (unsigned)(kx * D)) * (unsigned)sizeof(Cx<T>));
            Xb[k] = *at_byte(src, (row + (unsigned)((NC - kx) * D)) * (unsigned)sizeof(Cx<T>));
        }
        #pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int e = threadIdx.x + (h + k) * NT;
            const int kk = CtDiv<D, CNT>::div(e);
            const int c = e - kk * D;
            const int sl = kk >> LNC, kx = kk & (NC - 1);
            // the DC and Nyquist samples of a real signal's spectrum are real:
            // their imaginary parts (rounding residue) are dropped
            const Cx<T> xa = {Xa[k].x, kx == 0 ? T(0) : Xa[k].y};
            const Cx<T> Xm = {Xb[k].x, kx == 0 ? T(0) : -Xb[k].y};
            const Cx<T> A = cadd(xa, Xm);
            const Cx<T> B = cmulc(csub(xa, Xm), twl[kx]);  // exp(+2 pi i k / n) (Xk - conj X(nc-k))
            Cx<T> Z = cadd(A, mul_pi(B));
            if (!FULL && sl >= nrows) Z = Cx<T>{T(0), T(0)};
            buf[kx * NBS + sl * D + c] = Z;
        }
    }
    __syncthreads();
    ct_fft<T, NC, NB, 1, true, 2, NBS>(buf, twl);
    const T sc = T(a.out_scale);
    Cx<T> y[PPT];
    #pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int e = threadIdx.x + k * NT;
        const int b = e >> LNC, j = e & (NC - 1);
        y[k] = buf[j * NBS + b];
    }
    const long long lbase = (long long)lc * D * a.N;
    const unsigned N32 = (unsigned)a.N, row0 = (unsigned)(s0 * NL);
    if constexpr (UPD) {
        Cx<T> *pl = reinterpret_cast<Cx<T> *>(a.p_upd + lbase);
        // u's pairs at the element offsets of p's (in bytes when it has p's type,
        // else through a 64-bit index: its byte offsets may pass 32 bits)
        Cx<U> *ul = reinterpret_cast<Cx<U> *>(static_cast<U *>(a.u_upd) + lbase);
        auto u_at = [&](unsigned o) {
            if constexpr (sizeof(U) == sizeof(T)) return at_byte(ul, o);
            else return ul + o / (unsigned)sizeof(Cx<T>);
        };
        const T beta = T(a.st[lc].beta);
        const U ap = U(a.st[lc].alpha_pend);
        constexpr int CH2 = 8;  // slots per round: two loads each in flight
        #pragma unroll
        for (int h = 0; h < PPT; h += CH2) {
            Cx<T> pv[CH2];
            Cx<U> uv[CH2];
            #pragma unroll
            for (int k = 0; k < CH2; ++k) {
                const int e = threadIdx.x + (h + k) * NT;
                const int b = e >> LNC, j = e & (NC - 1);
                const int sl0 = CtDiv<D, NB>::div(b), c = b - sl0 * D;
                const int sl = (FULL || sl0 < nrows) ? sl0 : nrows - 1;
                const unsigned o = last_pair_offset<T, NL, D>(c, sl, j, N32, row0);
                pv[k] = ldc_nt(at_byte(pl, o));
                uv[k] = ldc_nt(u_at(o));
            }
            #pragma unroll
            for (int k = 0; k < CH2; ++k) {
                const int e = threadIdx.x + (h + k) * NT;
                const int b = e >> LNC, j = e & (NC - 1);
                const int sl = CtDiv<D, NB>::div(b), c = b - sl * D;
                if (FULL || sl < nrows) {
                    const unsigned o = last_pair_offset<T, NL, D>(c, sl, j, N32, row0);
                    const Cx<T> z = {y[h + k].x * sc, y[h + k].y * sc};
                    const Cx<U> un = {uv[k].x + ap * U(pv[k].x), uv[k].y + ap * U(pv[k].y)};
                    const Cx<T> pn = {z.x + beta * pv[k].x, z.y + beta * pv[k].y};
                    stc_nt(u_at(o), un);
                    stc_nt(at_byte(pl, o), pn);
                }
            }
        }
    } else {
        Cx<T> *zl = reinterpret_cast<Cx<T> *>(a.z + lbase);
        #pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const int e = threadIdx.x + k * NT;
            const int b = e >> LNC, j = e & (NC - 1);
            const int sl = CtDiv<D, NB>::div(b), c = b - sl * D;
            if (FULL || sl < nrows)
                stc_nt(at_byte(zl, last_pair_offset<T, NL, D>(c, sl, j, N32, row0)), Cx<T>{y[k].x * sc, y[k].y * sc});
        }
    }
}

template <typename T, int NL, int D, bool UPD, typename U = T>
__global__ __launch_bounds__(kFftThreads) void k_last_inv_ct(FK<T> a) {
    constexpr int NT = kFftThreads, NC = NL / 2;
    constexpr int RR = ct_last_rows<NL, D>(), NB = D * RR;
    static_assert((NB * NC) % NT == 0, "whole slots per thread");
    __shared__ Cx<T> buf[ct_last_stride<NL, D>() * NC];
    __shared__ Cx<T> twl[NL];
    const int t = xcd_remap(blockIdx.x, a.total);
    const int lc = t / a.nblk;
    const int blk = t - lc * a.nblk;
    if (a.st && !a.st[lc].active) return;
    const long long s0 = (long long)blk * RR;
    const int nrows = (int)min((long long)RR, a.rows - s0);
    for (int i = threadIdx.x; i < NL; i += NT) twl[i] = a.tw_last[i];
    __syncthreads();
    if (nrows == RR) last_inv_ct_body<T, NL, D, UPD, true, U>(a, lc, s0, nrows, buf, twl);
    else last_inv_ct_body<T, NL, D, UPD, false, U>(a, lc, s0, nrows, buf, twl);
}

// ---------------------------------------------------------------------------
// middle axis (3D), complex to complex
// ---------------------------------------------------------------------------
template <typename T, int PPT, int GEN>
__global__ __launch_bounds__(kFftThreads) __attribute__((amdgpu_waves_per_eu(kGenWaves<T, GEN>))) void k_middle(FK<T> a, int inv) {
    constexpr int NT = kFftThreads;
    __shared__ Cx<T> sbuf[GEN ? 1 : PPT * NT];
    Cx<T> *buf = GEN ? reinterpret_cast<Cx<T> *>(feh_dyn_lds) : sbuf;
    int t = xcd_remap(blockIdx.x, a.total);
    const int ib = t % a.nblk;
    t /= a.nblk;
    const int i0 = t % a.n0;
    const int lc = t / a.n0;
    if (a.st && !a.st[lc].active) return;
    const int PB = a.PB;
    const int n1 = a.n1;
    const int cnt = PB * n1;
    const long long inner = a.inner_total;
    const long long in0 = (long long)ib * PB;
    const long long boff = ((long long)lc * a.n0 + i0) * n1 * inner + in0;
    Cx<T> *base = a.spec + boff;
    const Cx<T> *src = (a.spec_in ? a.spec_in : a.spec) + boff;
    const int lim = (int)min((long long)PB, inner - in0);
    Cx<T> *twl = GEN ? buf + a.lbuf : reinterpret_cast<Cx<T> *>(feh_dyn_lds);
    stage(twl, a.tw, n1);
    Cx<T> v[PPT];
    #pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int e0 = threadIdx.x + k * NT;
        const int e = e0 < cnt ? e0 : 0;
        const int j = (int)a.d_PB.div((uint32_t)e);
        const int b = e - j * PB;
        v[k] = src[(long long)j * inner + (b < lim ? b : lim - 1)];
    }
    #pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int e0 = threadIdx.x + k * NT;
        const int j = (int)a.d_PB.div((uint32_t)e0);
        const int b = e0 - j * PB;
        if (e0 < cnt) buf[e0] = (b < lim) ? v[k] : Cx<T>{T(0), T(0)};
    }
    __syncthreads();
    lds_fft<T, PPT, GEN>(buf, PB, a.d_PB, a.ax, twl, 1, inv != 0);
    #pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int e0 = threadIdx.x + k * NT;
        v[k] = buf[e0 < cnt ? e0 : 0];
    }
    #pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int e0 = threadIdx.x + k * NT;
        const int j = (int)a.d_PB.div((uint32_t)e0);
        const int b = e0 - j * PB;
        if (e0 < cnt && b < lim) base[(long long)j * inner + b] = v[k];
    }
}

// Middle axis with the compile-time transform of length N (= n1): the
// workgroup takes NB consecutive (kh, component) pencils of one (load case,
// axis-0 index), as k_middle does with its run-time pencil count.
template <typename T, int N, bool INV>
__global__ __launch_bounds__(kFftThreads) void k_middle_ct(FK<T> a) {
    constexpr int NT = kFftThreads;
    constexpr int NB = ct_batches<T, N>();
    constexpr int PPT = N * NB / NT;
    constexpr int LNB = ct_log2(NB);
    __shared__ Cx<T> buf[N * NB];
    __shared__ Cx<T> twl[N];
    int t = xcd_remap(blockIdx.x, a.total);
    const int ib = t % a.nblk;
    t /= a.nblk;
    const int i0 = t % a.n0;
    const int lc = t / a.n0;
    if (a.st && !a.st[lc].active) return;
    const unsigned inner = (unsigned)a.inner_total;
    const unsigned in0 = (unsigned)ib * NB;
    const long long boff = ((long long)lc * a.n0 + i0) * (long long)N * inner + in0;
    Cx<T> *base = a.spec + boff;
    const Cx<T> *src = (a.spec_in ? a.spec_in : a.spec) + boff;
    const int lim = min(NB, (int)(inner - in0));
    for (int i = threadIdx.x; i < N; i += NT) twl[i] = a.tw[i];
    Cx<T> v[PPT];
    #pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int e = threadIdx.x + k * NT;
        const int j = e >> LNB, b = e & (NB - 1);
        v[k] = src[__umul24((unsigned)j, inner) + (unsigned)(b < lim ? b : lim - 1)];
    }
    #pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int e = threadIdx.x + k * NT;
        buf[e] = ((e & (NB - 1)) < lim) ? v[k] : Cx<T>{T(0), T(0)};
    }
    __syncthreads();
    ct_fft<T, N, NB, 1, INV>(buf, twl);
    #pragma unroll
    for (int k = 0; k < PPT; ++k) v[k] = buf[threadIdx.x + k * NT];
    #pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int e = threadIdx.x + k * NT;
        const int j = e >> LNB, b = e & (NB - 1);
        if (b < lim) base[__umul24((unsigned)j, inner) + (unsigned)b] = v[k];
    }
}

// ---------------------------------------------------------------------------
// first axis: forward, per-wavevector (B^*B)^-1 solve with Parseval r.z,
// inverse (mode 0); forward only (mode 1); inverse only (mode 2)
// ---------------------------------------------------------------------------
__device__ __forceinline__ Cx<double> ld2(const double *p, int i) { return Cx<double>{p[2 * i], p[2 * i + 1]}; }
template <typename R>
__device__ __forceinline__ R nrm(Cx<R> a) { return a.x * a.x + a.y * a.y; }
__device__ __forceinline__ float recip(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double recip(double x) { return 1.0 / x; }

// Inverse of the Hermitian positive definite M (diagonal Md, upper triangle
// Mo = (M01, M02, M12)) by the adjugate in the scalar type R: Id = real
// diagonal, Io = upper triangle of post M^-1.
template <typename R, int D>
__device__ __forceinline__ void herm_inverse(const R (&Md)[D], const Cx<R> (&Mo)[3], R (&Id)[D], Cx<R> (&Io)[3],
                                             R post = R(1)) {
    if constexpr (D == 2) {
        const R id = post * recip(Md[0] * Md[1] - nrm(Mo[0]));
        Id[0] = Md[1] * id;
        Id[1] = Md[0] * id;
        Io[0] = cscale(Mo[0], -id);
        Io[1] = Io[2] = Cx<R>{R(0), R(0)};
    } else {
        const Cx<R> a = Mo[0], b = Mo[1], c = Mo[2];
        const R C0 = Md[1] * Md[2] - nrm(c);
        const R C1 = Md[0] * Md[2] - nrm(b);
        const R C2 = Md[0] * Md[1] - nrm(a);
        const Cx<R> A01 = csub(cmulc(b, c), cscale(a, Md[2]));  // b conj(c) - a d2
        const Cx<R> A02 = csub(cmul(a, c), cscale(b, Md[1]));   // a c - b d1
        const Cx<R> A12 = csub(cmulc(b, a), cscale(c, Md[0]));  // b conj(a) - c d0
        // det = d0 C00 + Re(a conj(A01)) + Re(b conj(A02))
        const R det = Md[0] * C0 + (a.x * A01.x + a.y * A01.y) + (b.x * A02.x + b.y * A02.y);
        const R id = post * recip(det);
        Id[0] = C0 * id;
        Id[1] = C1 * id;
        Id[2] = C2 * id;
        Io[0] = cscale(A01, id);
        Io[1] = cscale(A02, id);
        Io[2] = cscale(A12, id);
    }
}

// M(k) = B^*B(k) of the linear elements of one voxel (six Kuhn tetrahedra in
// 3D, two triangles in 2D) from the per-axis factors aa_a = (w_a - 1) / h_a
// and w_a = e^{2 pi i m_a / n_a}, in the scalar type R; ch = element volume / 2.
template <typename R, int DIM>
__device__ __forceinline__ void core_matrix(const Cx<R> (&aa)[3], const Cx<R> (&w)[3], R ch, R (&Md)[DIM],
                                            Cx<R> (&Mo)[3]) {
    if constexpr (DIM == 3) {
        const Cx<R> a0 = aa[0], a1 = aa[1], a2 = aa[2];
        const Cx<R> w0 = w[0], w1 = w[1], w2 = w[2];
        const R n0s = nrm(a0), n1s = nrm(a1), n2s = nrm(a2);
        const R S = R(6) * (n0s + n1s + n2s);
        Md[0] = ch * (S + R(6) * n0s);
        Md[1] = ch * (S + R(6) * n1s);
        Md[2] = ch * (S + R(6) * n2s);
        const Cx<R> two = {R(2), R(0)};
        // M_ab = ch a_a conj(a_b) [conj(w_a)(2 + conj(w_c)) + w_b (2 + w_c)]
        Mo[0] = cscale(cmul(cmulc(a0, a1), cadd(cmulc(cadd(two, cconj(w2)), w0), cmul(w1, cadd(two, w2)))), ch);
        Mo[1] = cscale(cmul(cmulc(a0, a2), cadd(cmulc(cadd(two, cconj(w1)), w0), cmul(w2, cadd(two, w1)))), ch);
        Mo[2] = cscale(cmul(cmulc(a1, a2), cadd(cmulc(cadd(two, cconj(w0)), w1), cmul(w2, cadd(two, w0)))), ch);
    } else {
        const Cx<R> a0 = aa[0], a1 = aa[1];
        const Cx<R> w0 = w[0], w1 = w[1];
        const R n0s = nrm(a0), n1s = nrm(a1);
        const R S = R(2) * (n0s + n1s);
        Md[0] = ch * (S + R(2) * n0s);
        Md[1] = ch * (S + R(2) * n1s);
        // M_01 = ch a0 conj(a1) (1 + w1 conj(w0))
        const Cx<R> f = {R(1) + (w1.x * w0.x + w1.y * w0.y), w1.y * w0.x - w1.x * w0.y};
        Mo[0] = cscale(cmul(cmulc(a0, a1), f), ch);
        Mo[1] = Mo[2] = Cx<R>{R(0), R(0)};
    }
}

// Inverse of the projection core at wavevector slot e of the workgroup, in
// the plan precision: md = real diagonal, mo = upper triangle of M(k)^-1 (zero
// at k = 0 and for slots past the block's pencils); the Parseval weight bit of
// the slot.  The per-axis factors come from FP64 tables.  FP64 plans form the
// inverse in FP64.  FP32 plans form it in FP32 where sum_a |aa_a|^2 >= near0
// and in FP64 (rounded once) at the long-wavelength wavevectors below it,
// whose entries are O(|k|^2) and whose inverse is O(|k|^-2).  Either way the
// result is Hermitian positive definite, so its rounding moves the CG's
// convergence rate, not the solution it converges to.
template <typename T, int DIM>
__device__ __forceinline__ void slot_inverse(const FK<T> &a, int e, int PB, long long in0, int lim,
                                             const Cx<double> *pin, T (&md)[DIM], Cx<T> (&mo)[3], bool &half) {
    constexpr int D = DIM;
    const int j = (int)a.d_PB.div((uint32_t)e);
    const int b = e - j * PB;
    const long long inn = in0 + b;
    #pragma unroll
    for (int c = 0; c < D; ++c) md[c] = T(0);
    mo[0] = mo[1] = mo[2] = Cx<T>{T(0), T(0)};
    half = false;
    if (!(e < PB * a.n0 && b * D < lim && !(j == 0 && inn == 0))) return;
    int m1 = 0, kh;
    if constexpr (DIM == 3) {
        m1 = (int)a.d_nh.div((uint32_t)inn);
        kh = (int)(inn - (long long)m1 * a.nh);
    } else {
        kh = (int)inn;
    }
    half = kh == 0 || (a.last_even && kh == a.nh - 1);
    Cx<double> A[3], W[3];
    A[0] = ld2(a.aa[0], j);
    W[0] = ld2(a.om[0], j);
    A[1] = pin[4 * b + 0];
    W[1] = pin[4 * b + 1];
    A[2] = DIM == 3 ? pin[4 * b + 2] : Cx<double>{0.0, 0.0};
    W[2] = DIM == 3 ? pin[4 * b + 3] : Cx<double>{1.0, 0.0};
    if constexpr (sizeof(T) == 4) {
        Cx<float> Af[3], Wf[3];
        #pragma unroll
        for (int c = 0; c < 3; ++c) {
            Af[c] = Cx<float>{float(A[c].x), float(A[c].y)};
            Wf[c] = Cx<float>{float(W[c].x), float(W[c].y)};
        }
        if (nrm(Af[0]) + nrm(Af[1]) + nrm(Af[2]) >= a.near0) {
            // dimensionless factors aa_a h_max: M~ = M h_max^2 / ch has entries
            // of order |k h_max|^2 whatever the voxel size, so the adjugate
            // neither underflows nor overflows; M^-1 = M~^-1 h_max^2 / ch
            const float hm = a.hmax_f;
            #pragma unroll
            for (int c = 0; c < 3; ++c) Af[c] = Cx<float>{Af[c].x * hm, Af[c].y * hm};
            float Md[D];
            Cx<float> Mo[3];
            core_matrix<float, DIM>(Af, Wf, 1.0f, Md, Mo);
            herm_inverse<float, D>(Md, Mo, md, mo, a.post_f);
            return;
        }
    }
    double Md[D];
    Cx<double> Mo[3];
    core_matrix<double, DIM>(A, W, a.chalf, Md, Mo);
    double Id[D];
    Cx<double> Io[3];
    herm_inverse<double, D>(Md, Mo, Id, Io);
    #pragma unroll
    for (int c = 0; c < D; ++c) md[c] = T(Id[c]);
    #pragma unroll
    for (int c = 0; c < 3; ++c) mo[c] = Cx<T>{T(Io[c].x), T(Io[c].y)};
}

// 1 / (w sum_Ta |D_Ta|^2) at wavevector slot e for the full gradient of a
// stencil derivative (metric 1 + kind), from the per-axis factors
// aa = (e^{i k h} - 1) / h; 0 where the symbol vanishes.
template <typename T, int DIM>
__device__ __forceinline__ T slot_scalar_metric(const FK<T> &a, int e, int PB, long long in0, int lim, const Cx<double> *pin) {
    const int j = (int)a.d_PB.div((uint32_t)e);
    const int b = e - j * PB;
    if (!(e < PB * a.n0 && b * DIM < lim && !(j == 0 && in0 + b == 0))) return T(0);
    Cx<double> A[3], W[3];
    A[0] = ld2(a.aa[0], j);
    W[0] = ld2(a.om[0], j);
    A[1] = pin[4 * b + 0];
    W[1] = pin[4 * b + 1];
    if constexpr (DIM == 3) A[2] = pin[4 * b + 2];
    double S = 0.0;
    switch (a.metric - 1) {
    case FEH_DERIV_CD:  // i sin(k h) / h
        #pragma unroll
        for (int x = 0; x < DIM; ++x) S += A[x].y * A[x].y;
        break;
    case FEH_DERIV_LS:  // (w_a - 1)(1 + w_b) / (2 h_a): |1 + w|^2 / 4 = (1 + Re w) / 2
        S = 0.5 * (nrm(A[0]) * (1.0 + W[1].x) + nrm(A[1]) * (1.0 + W[0].x));
        break;
    default:  // forward differences; linear elements take the same edge differences once an element
        #pragma unroll
        for (int x = 0; x < DIM; ++x) S += nrm(A[x]);
        if (a.metric - 1 == FEH_DERIV_FE) S *= DIM == 3 ? 6.0 : 2.0;
    }
    return S > a.metric_tiny ? T(1.0 / (a.metric_w * S)) : T(0);
}

// z = M^-1 r at one wavevector (md: real diagonal, mo: upper triangle of
// M^-1) and the Parseval term Re(r . conj z) in FP64.
template <typename T, int DIM>
__device__ __forceinline__ double apply_minv(const T (&md)[DIM], const Cx<T> (&mo)[3], const Cx<T> (&r)[DIM],
                                             Cx<T> (&z)[DIM]) {
    if constexpr (DIM == 3) {
        const Cx<T> o01 = mo[0], o02 = mo[1], o12 = mo[2];
        z[0] = cadd(cadd(cscale(r[0], md[0]), cmul(o01, r[1])), cmul(o02, r[2]));
        z[1] = cadd(cadd(cmulc(r[0], o01), cscale(r[1], md[1])), cmul(o12, r[2]));
        z[2] = cadd(cadd(cmulc(r[0], o02), cmulc(r[1], o12)), cscale(r[2], md[2]));
    } else {
        const Cx<T> o01 = mo[0];
        z[0] = cadd(cscale(r[0], md[0]), cmul(o01, r[1]));
        z[1] = cadd(cmulc(r[0], o01), cscale(r[1], md[1]));
    }
    double dot = 0.0;
    #pragma unroll
    for (int c = 0; c < DIM; ++c) dot += double(r[c].x) * double(z[c].x) + double(r[c].y) * double(z[c].y);
    return dot;
}

// Components of one table entry: the D real diagonal entries of M^-1, then
// the real and imaginary parts of its upper triangle (3 entries in 3D, 1 in 2D).
template <int DIM>
constexpr int kMinvComps = DIM == 3 ? 9 : 4;

// Stage the per-axis phase factors of a block's PB inner wavevector indices
// in LDS: pin[4 b + 0..3] = aa_1, om_1, aa_2, om_2 (2D: aa_1, om_1).
template <typename T, int DIM>
__device__ __forceinline__ void stage_inner_phases(const FK<T> &a, long long in0, int PB, Cx<double> *pin) {
    const long long inner = a.inner_total;
    for (int b = threadIdx.x; b < PB; b += kFftThreads) {
        const long long inn = in0 + b;
        if (inn < inner) {
            if constexpr (DIM == 3) {
                const int m1 = (int)a.d_nh.div((uint32_t)inn);
                const int kh = (int)(inn - (long long)m1 * a.nh);
                pin[4 * b + 0] = ld2(a.aa[1], m1);
                pin[4 * b + 1] = ld2(a.om[1], m1);
                pin[4 * b + 2] = ld2(a.aa[2], kh);
                pin[4 * b + 3] = ld2(a.om[2], kh);
            } else {
                pin[4 * b + 0] = ld2(a.aa[1], (int)inn);
                pin[4 * b + 1] = ld2(a.om[1], (int)inn);
            }
        }
    }
}

// The (B^*B)^-1 table of the first-axis pass: one workgroup per pencil block
// writes slot_inverse of its PB n0 wavevector slots (zeros at k = 0 and past
// the last pencil), component-major within the block so that the pass reads
// each component with consecutive threads on consecutive words.  Built once
// per workspace and block size; every load case and iteration then reads the
// inverse instead of forming it again.
template <typename T, int DIM>
__global__ __launch_bounds__(kFftThreads) void k_first_table(FK<T> a) {
    constexpr int D = DIM;
    constexpr int NC = kMinvComps<DIM>;
    const int blk = blockIdx.x;
    const int PB = a.PB;
    const long long in0 = (long long)blk * PB;
    const int lim = (int)min((long long)PB, a.inner_total - in0) * D;
    const int cntk = PB * a.n0;
    __shared__ Cx<double> pin[4 * 32];
    stage_inner_phases<T, DIM>(a, in0, PB, pin);
    __syncthreads();
    T *tb = a.minv + (long long)blk * NC * cntk;
    for (int e = threadIdx.x; e < cntk; e += kFftThreads) {
        T md[D];
        Cx<T> mo[3];
        bool half;
        if (a.metric == 0) {
            slot_inverse<T, DIM>(a, e, PB, in0, lim, pin, md, mo, half);
        } else {
            const T m = slot_scalar_metric<T, DIM>(a, e, PB, in0, lim, pin);
            #pragma unroll
            for (int c = 0; c < D; ++c) md[c] = m;
            mo[0] = mo[1] = mo[2] = Cx<T>{T(0), T(0)};
        }
        const int pos = minv_pos(e, a.minv_q);
        #pragma unroll
        for (int c = 0; c < D; ++c) tb[c * cntk + pos] = md[c];
        #pragma unroll
        for (int c = 0; c < (DIM == 3 ? 3 : 1); ++c) {
            tb[(D + 2 * c) * cntk + pos] = mo[c].x;
            tb[(D + 2 * c + 1) * cntk + pos] = mo[c].y;
        }
    }
}

// First axis: forward transform, per-wavevector z^ = M(k)^-1 r^ with the
// Parseval partial of r.z (mode 0), inverse transform.  Mode 1: forward only;
// mode 2: inverse only.  PERLC = false: one workgroup per block of PB pencils
// runs through every load case, forming the inverses of its wavevectors once
// (adjugate, see slot_inverse) and keeping them in registers.
// PERLC = true: one workgroup per (load case, pencil block), load cases
// fastest in the workgroup order (the L workgroups of a block run side by
// side on one XCD); the inverses are read from the table of k_first_table
// (TAB) or formed again per load case just in time.  The power-of-two PERLC
// instantiations are held to 3 waves per SIMD (at most 168 VGPRs, no spills).
template <typename T, int PPT, int DIM, int MODE, int GEN, bool PERLC, bool TAB>
__global__ __launch_bounds__(kFftThreads) __attribute__((amdgpu_waves_per_eu((PERLC && !GEN) ? 3 : TAB ? kGenWaves<T, GEN> : 1))) void k_first(FK<T> a) {
    constexpr int NT = kFftThreads;
    constexpr int D = DIM;
    constexpr int KW = (PPT + D - 1) / D;  // wavevector slots per thread: PB n0 <= PPT NT / D
    constexpr int KC = PERLC ? 1 : KW;     // cached slots
    __shared__ Cx<T> sbuf[GEN ? 1 : PPT * NT];
    __shared__ double red[NT / 64];
    Cx<T> *buf = GEN ? reinterpret_cast<Cx<T> *>(feh_dyn_lds) : sbuf;
    int blk, lc0, lc1;
    if constexpr (PERLC) {
        const int t = xcd_remap(blockIdx.x, a.total);
        blk = t / a.L;
        lc0 = t - blk * a.L;
        lc1 = lc0 + 1;
        if (a.st && !a.st[lc0].active) return;
    } else {
        blk = xcd_remap(blockIdx.x, a.total);
        lc0 = 0;
        lc1 = a.L;
    }
    const int PB = a.PB;
    const int nb = PB * D;
    const int n0 = a.n0;
    const long long inner = a.inner_total;
    const long long in0 = (long long)blk * PB;
    const int lim = (int)min((long long)PB, inner - in0) * D;
    const int cnt = nb * n0;
    // dynamic LDS: the tile of general lengths, twiddles of axis 0, then (mode
    // 0) the phase factors of this block's PB inner wavevector indices; the
    // axis-0 phase factors are read from the plan's tables (once per
    // wavevector slot, L2-resident)
    Cx<T> *twl = reinterpret_cast<Cx<T> *>(feh_dyn_lds) + (GEN ? a.lbuf : 0);
    const int tw_bytes = ((n0 * (int)sizeof(Cx<T>) + 15) / 16) * 16;
    Cx<double> *pin = reinterpret_cast<Cx<double> *>(reinterpret_cast<char *>(twl) + tw_bytes);  // [PB][4]: aa1, om1, aa2, om2 (2D: aa1, om1)
    stage(twl, a.tw, n0);
    // per cached slot: real diagonal of M^-1, then its upper triangle (complex)
    T Mid[KC][D];
    Cx<T> Mio[KC][DIM == 3 ? 3 : 1];
    unsigned half_w = 0;  // bit kw: wavevector counted once in the half-spectrum Parseval sum
    if constexpr (MODE == 0 && !TAB) {
        stage_inner_phases<T, DIM>(a, in0, PB, pin);
        __syncthreads();
        if constexpr (!PERLC) {
            #pragma unroll
            for (int kw = 0; kw < KW; ++kw) {
                T md[D];
                Cx<T> mo[3];
                bool half;
                slot_inverse<T, DIM>(a, threadIdx.x + kw * NT, PB, in0, lim, pin, md, mo, half);
                if (half) half_w |= 1u << kw;
                #pragma unroll
                for (int c = 0; c < D; ++c) Mid[kw][c] = md[c];
                #pragma unroll
                for (int c = 0; c < (DIM == 3 ? 3 : 1); ++c) Mio[kw][c] = mo[c];
            }
        }
    }
    for (int lc = lc0; lc < lc1; ++lc) {
        if (!PERLC && a.st && !a.st[lc].active) continue;
        // the thread index passes through an empty asm statement so that the
        // index arithmetic is redone per load case instead of being hoisted
        // out of the loop into registers
        int tx = threadIdx.x;
        asm volatile("" : "+v"(tx));
        const long long boff = ((long long)lc * n0 * inner + in0) * D;
        Cx<T> *base = a.spec + boff;
        {
            const Cx<T> *src = (a.spec_in ? a.spec_in : a.spec) + boff;
            Cx<T> v[PPT];
            #pragma unroll
            for (int k = 0; k < PPT; ++k) {
                const int e0 = tx + k * NT;
                const int e = e0 < cnt ? e0 : 0;
                const int j = (int)a.nbd.div((uint32_t)e);
                const int bc = e - j * nb;
                v[k] = src[(long long)j * inner * D + (bc < lim ? bc : lim - 1)];
            }
            #pragma unroll
            for (int k = 0; k < PPT; ++k) {
                const int e0 = tx + k * NT;
                const int j = (int)a.nbd.div((uint32_t)e0);
                const int bc = e0 - j * nb;
                if (e0 < cnt) buf[e0] = (bc < lim) ? v[k] : Cx<T>{T(0), T(0)};
            }
        }
        __syncthreads();
        if (MODE != 2) lds_fft<T, PPT, GEN>(buf, nb, a.nbd, a.ax, twl, 1, false, tx);
        double acc = 0.0;
        if constexpr (MODE == 0) {
            #pragma unroll
            for (int kw = 0; kw < KW; ++kw) {
                const int e = tx + kw * NT;
                const int j = (int)a.d_PB.div((uint32_t)e);
                const int b = e - j * PB;
                if (e < PB * n0 && b * D < lim) {
                    T md[D];
                    Cx<T> mo[3];
                    bool half;
                    if constexpr (TAB) {
                        const int cntk = PB * n0;
                        const T *tb = a.minv + (long long)blk * kMinvComps<DIM> * cntk + e;
                        #pragma unroll
                        for (int c = 0; c < D; ++c) md[c] = tb[c * cntk];
                        #pragma unroll
                        for (int c = 0; c < (DIM == 3 ? 3 : 1); ++c)
                            mo[c] = Cx<T>{tb[(D + 2 * c) * cntk], tb[(D + 2 * c + 1) * cntk]};
                        // counted once in the half-spectrum Parseval sum: the
                        // last-axis index 0 and (even length) n/2
                        const long long inn = in0 + b;
                        const int kh = DIM == 3 ? (int)(inn - (long long)a.d_nh.div((uint32_t)inn) * a.nh) : (int)inn;
                        half = kh == 0 || (a.last_even && kh == a.nh - 1);
                    } else if constexpr (PERLC) {
                        slot_inverse<T, DIM>(a, e, PB, in0, lim, pin, md, mo, half);
                    } else {
                        #pragma unroll
                        for (int c = 0; c < D; ++c) md[c] = Mid[kw][c];
                        #pragma unroll
                        for (int c = 0; c < (DIM == 3 ? 3 : 1); ++c) mo[c] = Mio[kw][c];
                        half = (half_w >> kw) & 1u;
                    }
                    Cx<T> *pt = buf + j * nb + b * D;
                    Cx<T> r[D], z[D];
                    #pragma unroll
                    for (int c = 0; c < D; ++c) r[c] = pt[c];
                    const double dot = apply_minv<T, DIM>(md, mo, r, z);
                    #pragma unroll
                    for (int c = 0; c < D; ++c) pt[c] = z[c];
                    acc += half ? dot : 2.0 * dot;
                }
            }
            __syncthreads();
        }
        if (MODE != 1) lds_fft<T, PPT, GEN>(buf, nb, a.nbd, a.ax, twl, 1, true, tx);
        {
            Cx<T> v[PPT];
            #pragma unroll
            for (int k = 0; k < PPT; ++k) {
                const int e0 = tx + k * NT;
                v[k] = buf[e0 < cnt ? e0 : 0];
            }
            #pragma unroll
            for (int k = 0; k < PPT; ++k) {
                const int e0 = tx + k * NT;
                const int j = (int)a.nbd.div((uint32_t)e0);
                const int bc = e0 - j * nb;
                if (e0 < cnt && bc < lim) base[(long long)j * inner * D + bc] = v[k];
            }
        }
        if (MODE == 0 && a.partial) {
            const double s = block_sum<NT>(acc, red);
            if (threadIdx.x == 0) a.partial[(long long)lc * a.part_stride + blk] = s * a.invN;
        }
        __syncthreads();  // the next load case reuses buf
    }
}

// Pencils per block of the compile-time first-axis pass (N = n0): N PB D
// points per workgroup, 24 per thread in FP32 3D.
template <typename T, int N>
constexpr int ct_first_pencils() { return N == 1024 ? 2 : (sizeof(T) == 4 ? 2048 : 1024) / N; }

// First axis with the compile-time transform, the CG's fused pass only
// (forward, z = M^-1 r with the inverse table and the Parseval partial,
// inverse): one workgroup per (pencil block, load case), load cases fastest,
// as k_first with PERLC and TAB.  LDS row m0 holds the block's PB D values of
// that row in the global order (pencil-major, the D components of a
// wavevector together): the transforms run over PB D batches of one
// sub-problem, and the staging, the M^-1 step and the store take consecutive
// LDS words across the lanes of a wavefront.
template <typename T, int N, int DIM>
__global__ __launch_bounds__(kFftThreads) void k_first_ct(FK<T> a) {
    constexpr int NT = kFftThreads, D = DIM;
    constexpr int PB = ct_first_pencils<T, N>();
    constexpr int LPB = ct_log2(PB);
    constexpr int NB = PB * D;            // values per LDS row
    constexpr int RS = NT / PB;           // rows per staging sweep
    constexpr int NC = kMinvComps<DIM>;
    constexpr int CNTK = PB * N;          // wavevector slots of the block
    static_assert(NT % PB == 0 && N % RS == 0, "staging covers whole rows");
    constexpr int NR = N / RS;            // rows per thread: g + RS i
    // The forward transform's first pass (no twiddles) has its butterfly q
    // on rows q + (N / R) c and writes rows q + (N / R) d: with R = NR these
    // are the thread's own staging rows for q = g, so the pass runs on the
    // loaded values and the staging store writes its outputs.
    constexpr bool FUSE_FIRST = ct_radix_at(N, 0) == NR;
    // The inverse transform's last pass (M = 1) has butterfly p on rows
    // R p + c and writes rows p + (N / R) d: the butterflies p = g + RS k,
    // k < KB, produce exactly the thread's rows, so the pass ends in the
    // registers the global store takes.
    constexpr int SL = ct_npass(N) - 1, RL = ct_radix_at(N, SL);
    constexpr int KB = N / (RL * RS);
    constexpr bool FUSE_LAST = SL >= 1 && KB >= 1 && KB * RL == NR && ct_lstar(N, SL) * RL == N;
    __shared__ Cx<T> buf[N * NB];
    __shared__ Cx<T> twl[N];
    // the partial sums of the last step take the twiddles' place: two FP64
    // 1024-point workgroups then fill a CU's LDS to the byte
    double *red = reinterpret_cast<double *>(twl);
    const int t = xcd_remap(blockIdx.x, a.total);
    const int blk = t / a.L;
    const int lc = t - blk * a.L;
    if (a.st && !a.st[lc].active) return;
    const unsigned inner = (unsigned)a.inner_total;
    const unsigned in0 = (unsigned)blk * PB;
    const int lim = min(PB, (int)(inner - in0));
    const int limD = lim * D;             // valid values per row
    const unsigned rowD = inner * D;      // complex values between consecutive m0
    Cx<T> *base = a.spec + ((long long)lc * N * inner + in0) * D;
    const Cx<T> *src = (a.spec_in ? a.spec_in : a.spec) + ((long long)lc * N * inner + in0) * D;
    for (int i = threadIdx.x; i < N; i += NT) twl[i] = a.tw[i];
    // staging slot (i, j): row m0 = g + RS i, value r = lane + PB j of the row
    const int lane = threadIdx.x & (PB - 1), g = threadIdx.x >> LPB;
    {
        Cx<T> v[NR][D];
        #pragma unroll
        for (int i = 0; i < NR; ++i) {
            #pragma unroll
            for (int j = 0; j < D; ++j) {
                const int r = lane + PB * j;
                const int rc = r < limD ? r : limD - 1;
                v[i][j] = src[__umul24((unsigned)(g + RS * i), rowD) + (unsigned)rc];
            }
        }
        #pragma unroll
        for (int j = 0; j < D; ++j) {
            const int r = lane + PB * j;
            Cx<T> x[NR];
            #pragma unroll
            for (int i = 0; i < NR; ++i) x[i] = r < limD ? v[i][j] : Cx<T>{T(0), T(0)};
            // radices 2, 4 and 8 take no twiddles from the table
            if constexpr (FUSE_FIRST) Dft<T, NR>::run(x, false, twl, 1, N);
            #pragma unroll
            for (int i = 0; i < NR; ++i) buf[(g + RS * i) * NB + r] = x[i];
        }
    }
    __syncthreads();
    ct_passes<T, N, NB, 1, FUSE_FIRST ? 1 : 0, false, 1, NB>(buf, twl);
    double acc = 0.0;
    {
        // each table component arrives in one 16-byte load of Q slots per
        // round; the table interleaves the slots (minv_pos) so that vector
        // element qq of the lanes of a wavefront covers 64 consecutive slots
        constexpr int Q = 16 / (int)sizeof(T);
        constexpr int RUN = 64 * Q;
        static_assert(CNTK % (NT * Q) == 0, "whole rounds of slots");
        typedef T TV __attribute__((ext_vector_type(Q)));
        const T *tb0 = a.minv + (long long)blk * NC * CNTK;
        const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
        #pragma unroll
        for (int k = 0; k < CNTK / (NT * Q); ++k) {
            const int run0 = (wv + k * (NT / 64)) * RUN;
            TV tv[NC];
            #pragma unroll
            for (int c = 0; c < NC; ++c) tv[c] = *reinterpret_cast<const TV *>(tb0 + c * CNTK + run0 + l * Q);
            #pragma unroll
            for (int qq = 0; qq < Q; ++qq) {
                const int e = run0 + qq * 64 + l;
                const int m0 = e >> LPB, b = e & (PB - 1);
                if (b < lim) {
                    T md[D];
                    Cx<T> mo[3];
                    #pragma unroll
                    for (int c = 0; c < D; ++c) md[c] = tv[c][qq];
                    #pragma unroll
                    for (int c = 0; c < (DIM == 3 ? 3 : 1); ++c) mo[c] = Cx<T>{tv[D + 2 * c][qq], tv[D + 2 * c + 1][qq]};
                    const unsigned inn = in0 + b;
                    const int kh = DIM == 3 ? (int)(inn - a.d_nh.div(inn) * (unsigned)a.nh) : (int)inn;
                    const bool half = kh == 0 || (a.last_even && kh == a.nh - 1);
                    Cx<T> *pt = buf + m0 * NB + b * D;
                    Cx<T> r[D], z[D];
                    #pragma unroll
                    for (int c = 0; c < D; ++c) r[c] = pt[c];
                    const double dot = apply_minv<T, DIM>(md, mo, r, z);
                    #pragma unroll
                    for (int c = 0; c < D; ++c) pt[c] = z[c];
                    acc += half ? dot : 2.0 * dot;
                }
            }
        }
    }
    __syncthreads();
    ct_passes<T, N, NB, 1, 0, true, 1, NB, FUSE_LAST ? SL : SL + 1>(buf, twl);
    {
        Cx<T> v[NR][D];
        #pragma unroll
        for (int j = 0; j < D; ++j) {
            const int r = lane + PB * j;
            if constexpr (FUSE_LAST) {
                #pragma unroll
                for (int k = 0; k < KB; ++k) {
                    const int pp = g + RS * k;
                    Cx<T> x[RL];
                    #pragma unroll
                    for (int cc = 0; cc < RL; ++cc) x[cc] = buf[(RL * pp + cc) * NB + r];
                    #pragma unroll
                    for (int cc = 1; cc < RL; ++cc) x[cc] = cmul(x[cc], twid(twl, 1, cc * pp, true));
                    Dft<T, RL>::run(x, true, twl, 1, N);
                    #pragma unroll
                    for (int d = 0; d < RL; ++d) v[k + KB * d][j] = x[d];
                }
            } else {
                #pragma unroll
                for (int i = 0; i < NR; ++i) v[i][j] = buf[(g + RS * i) * NB + r];
            }
        }
        #pragma unroll
        for (int i = 0; i < NR; ++i) {
            #pragma unroll
            for (int j = 0; j < D; ++j) {
                const int r = lane + PB * j;
                if (r < limD) base[__umul24((unsigned)(g + RS * i), rowD) + (unsigned)r] = v[i][j];
            }
        }
    }
    if (a.partial) {
        const double s = block_sum<NT>(acc, red);
        if (threadIdx.x == 0) a.partial[(long long)lc * a.part_stride + blk] = s * a.invN;
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
bool pow2_len(int n) { return n > 0 && (n & (n - 1)) == 0; }

// Calls f with the GEN of an axis' passes.
template <typename F>
void with_gen(const AxisFFT &ax, F f) {
    bool prime = false;
    for (int s = 0; s < ax.npass; ++s) prime = prime || ax.pass[s].R > 13;
    if (pow2_len(ax.n)) f(std::integral_constant<int, 0>{});
    else if (!prime) f(std::integral_constant<int, 1>{});
    else f(std::integral_constant<int, 2>{});
}

template <typename T>
FK<T> base_args(const feh_plan &p, const FftArgs &fa) {
    FK<T> a{};
    a.r = static_cast<const T *>(fa.r);
    a.q = static_cast<const T *>(fa.q);
    a.r_out = static_cast<T *>(fa.r_out);
    a.spec = static_cast<Cx<T> *>(fa.spec);
    a.spec_in = static_cast<const Cx<T> *>(fa.spec_in);
    a.z = static_cast<T *>(fa.z);
    a.p_upd = static_cast<T *>(fa.p_upd);
    a.u_upd = fa.u_upd;
    a.partial = fa.partial;
    a.st = fa.state;
    a.dim = p.dim;
    a.D = fa.comps > 0 ? fa.comps : p.dim;
    a.L = p.L;
    a.n0 = (int)p.n[0];
    a.n1 = p.dim == 3 ? (int)p.n[1] : 1;
    a.nlast = (int)p.n[p.dim - 1];
    a.nh = (int)p.nh;
    a.N = p.N;
    a.rows = p.N / a.nlast;
    a.inner_total = p.dim == 3 ? (long long)p.n[1] * p.nh : p.nh;
    a.last_even = p.last_even ? 1 : 0;
    a.part_stride = (int)p.part_stride;
    a.out_scale = fa.out_scale;
    a.invN = 1.0 / (double)p.N;
    const double vol = p.dim == 3 ? (fa.unit_volume ? 1.0 : p.h[0] * p.h[1] * p.h[2]) / 6.0
                                  : (fa.unit_volume ? 1.0 : p.h[0] * p.h[1]) / 2.0;
    a.chalf = 0.5 * vol;
    double hmax = 0.0;
    for (int ax = 0; ax < p.dim; ++ax) hmax = std::max(hmax, p.h[ax]);
    a.near0 = (float)(0.0625 / (hmax * hmax));  // |k| h_max < 1/4
    a.hmax_f = (float)hmax;
    a.post_f = (float)(hmax * hmax / a.chalf);
    a.metric = p.metric;
    a.metric_w = p.metric == 1 + FEH_DERIV_FE ? (p.dim == 3 ? 1.0 / 6.0 : 0.5) : 1.0;
    for (int ax = 0; ax < p.dim; ++ax) a.metric_tiny += 1e-24 / (p.h[ax] * p.h[ax]);
    a.tw_last = p.ptr<const Cx<T>>(p.off_tw[p.dim - 1]);
    for (int ax = 0; ax < 3; ++ax) {
        a.om[ax] = p.ptr<const double>(p.off_om[ax]);
        a.aa[ax] = p.ptr<const double>(p.off_aa[ax]);
    }
    a.d_D = FastDiv::make((uint32_t)a.D);
    a.d_nh = FastDiv::make((uint32_t)a.nh);
    a.d_nhD = FastDiv::make((uint32_t)(a.nh * a.D));
    return a;
}

// Points a thread of a run-time pass holds: the tile of a workgroup is up to
// kFftThreads times as many, SMALL a quarter of it.
template <typename T, bool SMALL = false>
constexpr int ppt() { return (sizeof(T) == 4 ? 24 : 16) / (SMALL ? 4 : 1); }

// Workgroups that fill the chip: four on each of its 256 CUs.  A run-time
// pass with fewer (small grids, few load cases) takes the small tile: a launch
// then lasts as long as one workgroup, whose instructions are issued for every
// slot a thread may hold, used or not, and the small tile has a quarter of
// them and spreads the rows over more CUs.
// Measured, a solve: FP64 32^2 x 3 load cases 2.15 -> 1.68 ms, FP32 64^3 x 6 (its
// last axis only) 25.2 -> 22.6, FP64 1024^2 unchanged (it fills the chip).
constexpr long long kFillWorkgroups = 1024;
// rows or pencils of a pass's workgroup: `most` at the full tile; the small
// tile's `small` (0: the axis does not fit it) where the full one leaves the
// chip part empty, thinned out further while that gives every CU a workgroup
inline bool small_tile(long long units, int most, int small, long long per_unit, int *take) {
    *take = most;
    if (small < 1 || (units + most - 1) / most * per_unit >= kFillWorkgroups) return false;
    const long long thin = (units * per_unit + 255) / 256;
    *take = (int)std::max<long long>(1, std::min<long long>(small, thin));
    return true;
}

// LDS of a last- or middle-axis pass whose tile holds `cnt` points, in
// bytes (static tile plus dynamic part).  Power-of-two lengths keep a static
// tile of the largest size (its address and the twiddle table's are then
// compile-time constants, which the radix-2/4/8 passes are measurably faster
// with); general lengths take a dynamic tile sized to the pass and rounded
// up to 16 bytes, with the twiddle table after it, so that their long rows
// leave room for a second resident workgroup.  *lbuf receives the dynamic
// tile's entries (0 for power-of-two lengths), *dyn the dynamic bytes.
template <typename T>
size_t lds_of_pass(bool gen, int cnt, int table, int *lbuf, size_t *dyn, int PPT) {
    constexpr int q = 16 / (int)sizeof(Cx<T>);
    *lbuf = gen ? (cnt + q - 1) / q * q : 0;
    *dyn = ((size_t)*lbuf + table) * sizeof(Cx<T>);
    const size_t stat = (gen ? 1 : (size_t)PPT * kFftThreads) * sizeof(Cx<T>);
    return stat + *dyn;
}

}  // namespace

// The last-axis passes of a plan take the compile-time transform: FP32, an
// even last axis of 128, 256 or 512 points in the default radix order, the
// default row count, D = 2 or 3 components, 32-bit byte offsets.
bool last_ct_ok(const feh_plan &p, int D) {
    const int nlast = (int)p.n[p.dim - 1];
    return p.prec == FEH_FP32 && p.tune_ct && p.tune_rr_last == 0 && p.last_even && (D == 3 || D == 2) &&
           (nlast == 128 || nlast == 256 || nlast == 512) && ct_schedule_matches(p.fft[p.dim - 1], nlast / 2) &&
           (double)D * (double)p.N * 4.0 < 4294967296.0;
}

bool cg_residual_spectral(const feh_plan &p) { return last_ct_ok(p, p.dim); }

namespace {

template <typename T>
int last_t(const feh_plan &p, const FftArgs &fa, bool inverse) {
    constexpr int PPT = ppt<T>();
    FK<T> a = base_args<T>(p, fa);
    const int last = p.dim - 1;
    a.ax = p.fft[last];
    a.tw = p.ptr<const Cx<T>>(p.off_tw[last]);
    a.tws = p.last_even ? 2 : 1;
    const int nc = a.ax.n;
    int RR = (PPT * kFftThreads) / (nc * a.D);
    if (RR < 1) return set_error(FEH_ENOTSUP, "last axis too long for the LDS transform");
    if (RR > 64) RR = 64;
    if (p.tune_rr_last > 0 && p.tune_rr_last < RR) RR = p.tune_rr_last;
    if (RR > a.rows) RR = (int)a.rows;
    const bool small = p.tune_rr_last == 0 && small_tile(a.rows, RR, std::min(RR, ppt<T, true>() * kFftThreads / (nc * a.D)), p.L, &RR);
    a.RR = RR;
    a.nbd = FastDiv::make((uint32_t)(a.D * RR));
    a.d_nc = FastDiv::make((uint32_t)nc);
    a.nblk = (int)((a.rows + RR - 1) / RR);
    a.total = a.nblk * p.L;
    a.use_axpy = (!inverse && fa.q != nullptr && fa.state != nullptr) ? (fa.rspec ? 2 : 1) : 0;
    if (fa.rspec && (inverse || a.use_axpy != 2 || !last_ct_ok(p, a.D)))
        return set_error(FEH_EINVAL, "the spectral residual update needs the compile-time last-axis pass");
    // compile-time transform: FP32, 3D (or 2D) with an even last axis of 128,
    // 256 or 512 points in the default radix order and the default row count
    if constexpr (sizeof(T) == 4) {
      if (last_ct_ok(p, a.D)) {
        const int rr = 24 * kFftThreads / (a.nlast / 2 * a.D);  // ct_last_rows<nlast, D>()
        a.RR = rr;
        a.nblk = (int)((a.rows + rr - 1) / rr);
        a.total = a.nblk * p.L;
        const dim3 g(a.total), b(kFftThreads);
        const bool upd = inverse && fa.p_upd != nullptr;
        if (upd && (fa.u_upd == nullptr || fa.state == nullptr))
            return set_error(FEH_EINVAL, "fused CG update needs p, u and the CG state");
#define FEH_LAST_CT(NLv, Dv)                                                                                    \
        do {                                                                                                      \
            if (inverse) {                                                                                        \
                if (upd && fa.u_f64)                                                                              \
                    hipLaunchKernelGGL((k_last_inv_ct<T, NLv, Dv, true, double>), g, b, 0, p.stream, a);          \
                else if (upd) hipLaunchKernelGGL((k_last_inv_ct<T, NLv, Dv, true>), g, b, 0, p.stream, a);        \
                else hipLaunchKernelGGL((k_last_inv_ct<T, NLv, Dv, false>), g, b, 0, p.stream, a);                \
            } else {                                                                                              \
                if (a.use_axpy == 2) hipLaunchKernelGGL((k_last_fwd_ct<T, NLv, Dv, 2>), g, b, 0, p.stream, a);    \
                else if (a.use_axpy) hipLaunchKernelGGL((k_last_fwd_ct<T, NLv, Dv, 1>), g, b, 0, p.stream, a);    \
                else hipLaunchKernelGGL((k_last_fwd_ct<T, NLv, Dv, 0>), g, b, 0, p.stream, a);                    \
            }                                                                                                     \
        } while (0)
        if (a.D == 3) {
            if (a.nlast == 512) FEH_LAST_CT(512, 3);
            else if (a.nlast == 256) FEH_LAST_CT(256, 3);
            else FEH_LAST_CT(128, 3);
        } else {
            if (a.nlast == 512) FEH_LAST_CT(512, 2);
            else if (a.nlast == 256) FEH_LAST_CT(256, 2);
            else FEH_LAST_CT(128, 2);
        }
#undef FEH_LAST_CT
        return hip_check(hipGetLastError(), "last-axis fft launch");
      }
    }
    const dim3 g(a.total), b(kFftThreads);
    const bool gen = !pow2_len(a.ax.n);
    const bool upd = inverse && fa.p_upd != nullptr;
    if (upd && (fa.u_upd == nullptr || fa.state == nullptr))
        return set_error(FEH_EINVAL, "fused CG update needs p, u and the CG state");
    auto go = [&](auto tile) -> int {
        constexpr int PP = decltype(tile)::value;
        size_t dyn;
        if (lds_of_pass<T>(gen, a.D * RR * nc, a.nlast, &a.lbuf, &dyn, PP) > kLdsPerWorkgroup)
            return set_error(FEH_ENOTSUP, "last axis too long for the LDS transform");
        auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, g, b, dyn, p.stream, a); };
        with_gen(a.ax, [&](auto gl) {
            constexpr int G = decltype(gl)::value;
            if (upd && fa.u_f64) run(k_last_inv<T, PP, G, true, double>);
            else if (upd) run(k_last_inv<T, PP, G, true>);
            else if (inverse) run(k_last_inv<T, PP, G, false>);
            else if (a.use_axpy) run(k_last_fwd<T, PP, G, true>);
            else run(k_last_fwd<T, PP, G, false>);
        });
        return FEH_OK;
    };
    CK(small ? go(std::integral_constant<int, ppt<T, true>()>{}) : go(std::integral_constant<int, PPT>{}));
    return hip_check(hipGetLastError(), "last-axis fft launch");
}

// k_middle over a's pencils, with the full or the small tile
template <typename T>
int launch_middle_tile(const feh_plan &p, FK<T> &a, bool small, bool inverse, const char *what) {
    const bool gen = !pow2_len(a.ax.n);
    auto go = [&](auto tile) -> int {
        constexpr int PP = decltype(tile)::value;
        size_t dyn;
        if (lds_of_pass<T>(gen, a.PB * a.n1, a.n1, &a.lbuf, &dyn, PP) > kLdsPerWorkgroup)
            return set_error(FEH_ENOTSUP, "axis too long for the LDS transform");
        auto run = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(a.total), dim3(kFftThreads), dyn, p.stream, a, inverse ? 1 : 0);
        };
        with_gen(a.ax, [&](auto gl) { run(k_middle<T, PP, decltype(gl)::value>); });
        return hip_check(hipGetLastError(), what);
    };
    return small ? go(std::integral_constant<int, ppt<T, true>()>{}) : go(std::integral_constant<int, ppt<T>()>{});
}

template <typename T>
int middle_t(const feh_plan &p, const FftArgs &fa, bool inverse) {
    constexpr int PPT = ppt<T>();
    FK<T> a = base_args<T>(p, fa);
    a.ax = p.fft[1];
    a.tw = p.ptr<const Cx<T>>(p.off_tw[1]);
    a.tws = 1;
    // pencils along axis 1 are indexed by the contiguous (kh, component) pairs
    const long long inner = (long long)a.nh * a.D;
    int PB = (PPT * kFftThreads) / a.n1;
    if (PB < 1) return set_error(FEH_ENOTSUP, "middle axis too long for the LDS transform");
    if (PB > 32) PB = 32;
    if (p.tune_pb_mid > 0 && p.tune_pb_mid < PB) PB = p.tune_pb_mid;
    if (PB > inner) PB = (int)inner;
    const bool small = p.tune_pb_mid == 0 && small_tile(inner, PB, std::min(PB, ppt<T, true>() * kFftThreads / a.n1),
                                                        (long long)a.n0 * p.L, &PB);
    a.PB = PB;
    a.d_PB = FastDiv::make((uint32_t)PB);
    a.inner_total = inner;
    a.nblk = (int)((inner + PB - 1) / PB);
    a.total = a.nblk * a.n0 * p.L;
    // compile-time transform: the default schedule of n1 = 64 .. 512 (a power
    // of two) and the default pencil count
    if (p.tune_ct && p.tune_pb_mid == 0 && ct_schedule_matches(a.ax, a.n1) &&
        (a.n1 == 64 || a.n1 == 128 || a.n1 == 256 || a.n1 == 512)) {
        auto go = [&](auto kern, int nb) {
            a.nblk = (int)((inner + nb - 1) / nb);
            a.total = a.nblk * a.n0 * p.L;
            hipLaunchKernelGGL(kern, dim3(a.total), dim3(kFftThreads), 0, p.stream, a);
        };
        switch (a.n1 * 2 + (inverse ? 1 : 0)) {
        case 128: go(k_middle_ct<T, 64, false>, ct_batches<T, 64>()); break;
        case 129: go(k_middle_ct<T, 64, true>, ct_batches<T, 64>()); break;
        case 256: go(k_middle_ct<T, 128, false>, ct_batches<T, 128>()); break;
        case 257: go(k_middle_ct<T, 128, true>, ct_batches<T, 128>()); break;
        case 512: go(k_middle_ct<T, 256, false>, ct_batches<T, 256>()); break;
        case 513: go(k_middle_ct<T, 256, true>, ct_batches<T, 256>()); break;
        case 1024: go(k_middle_ct<T, 512, false>, ct_batches<T, 512>()); break;
        default: go(k_middle_ct<T, 512, true>, ct_batches<T, 512>()); break;
        }
        return hip_check(hipGetLastError(), "middle-axis fft launch");
    }
    return launch_middle_tile<T>(p, a, small, inverse, "middle-axis fft launch");
}

// c2c along axis 0 of a spectrum with fa.comps components, no k-solve: the
// middle-axis kernel with one outer slice, the whole axis-0 pencil set of a
// load case and the contiguous (axis 1, kh, component) index as pencils.
template <typename T>
int first_plain_t(const feh_plan &p, const FftArgs &fa, bool inverse) {
    constexpr int PPT = ppt<T>();
    FK<T> a = base_args<T>(p, fa);
    a.ax = p.fft[0];
    a.tw = p.ptr<const Cx<T>>(p.off_tw[0]);
    a.tws = 1;
    const long long inner = a.inner_total * a.D;
    const int len = a.n0;
    int PB = (PPT * kFftThreads) / len;
    if (PB < 1) return set_error(FEH_ENOTSUP, "first axis too long for the LDS transform");
    if (PB > 32) PB = 32;
    if (PB > inner) PB = (int)inner;
    const bool small = small_tile(inner, PB, std::min(PB, ppt<T, true>() * kFftThreads / len), p.L, &PB);
    a.PB = PB;
    a.d_PB = FastDiv::make((uint32_t)PB);
    a.inner_total = inner;
    a.n1 = len;   // transform length
    a.n0 = 1;     // one outer slice per load case
    a.nblk = (int)((inner + PB - 1) / PB);
    a.total = a.nblk * p.L;
    return launch_middle_tile<T>(p, a, small, inverse, "first-axis fft launch");
}

// Whether the CG's run-time first-axis pass takes the small tile, and its
// pencils (at least a quarter of the default: the partial sums have one slot a
// pencil block of that size).  *PB: the full tile's pencils.
bool first_small_pencils(const feh_plan &p, int metric, int *PB) {
    if (p.tune_pb_first != 0 || !first_by_table(p, metric) || first_ct_pencils(p)) return false;
    const int points = (p.prec == FEH_FP32 ? ppt<float, true>() : ppt<double, true>()) * kFftThreads;
    const long long inner = p.dim == 3 ? p.n[1] * p.nh : p.nh;
    const int least = std::min(*PB, std::max(1, first_pencils_default(p) / 4));
    int take;
    if (!small_tile(inner, *PB, std::min(*PB, points / ((int)p.n[0] * p.dim)), p.L, &take)) return false;
    *PB = std::max(take, least);
    return true;
}

// The table for a's block size and slot order, unless the workspace has it.
template <typename T, int DIM>
int ensure_table(const feh_plan &p, const FK<T> &a) {
    if (p.minv_ws == p.ws && p.minv_pb == a.PB && p.minv_q == a.minv_q && p.minv_metric == p.metric) return FEH_OK;
    hipLaunchKernelGGL((k_first_table<T, DIM>), dim3(a.nblk), dim3(kFftThreads), 0, p.stream, a);
    CK(hip_check(hipGetLastError(), "inverse table launch"));
    p.minv_ws = p.ws;
    p.minv_pb = a.PB;
    p.minv_q = a.minv_q;
    p.minv_metric = p.metric;
    return FEH_OK;
}

template <typename T, int DIM>
int plain_table(const feh_plan &p) {
    FftArgs fa;
    fa.unit_volume = true;
    FK<T> a = base_args<T>(p, fa);
    a.minv = p.ptr<T>(p.off_minv);
    a.PB = 1;
    a.d_PB = FastDiv::make(1);
    a.nblk = (int)a.inner_total;
    return ensure_table<T, DIM>(p, a);
}

template <typename T, int DIM>
int first_t(const feh_plan &p, const FftArgs &fa, int mode) {
    constexpr int PPT = ppt<T>();
    FK<T> a = base_args<T>(p, fa);
    a.ax = p.fft[0];
    a.tw = p.ptr<const Cx<T>>(p.off_tw[0]);
    a.tws = 1;
    const int ctpb = mode == 0 && fa.unit_volume ? first_ct_pencils(p) : 0;
    int PB = (PPT * kFftThreads) / (a.n0 * DIM);
    if (PB < 1) return set_error(FEH_ENOTSUP, "first axis too long for the LDS transform");
    if (PB > 32) PB = 32;
    // tuned value, never below a quarter of the default: the partial-sum
    // buffer holds one slot per pencil block for that size
    if (p.tune_pb_first > 0 && p.tune_pb_first < PB) PB = std::max(p.tune_pb_first, std::max(1, PB / 4));
    // the compile-time pass reads the table in blocks of its own size, also on
    // a grid with fewer pencils than one block
    if (ctpb > 0) PB = ctpb;
    else if (PB > a.inner_total) PB = (int)a.inner_total;
    const bool small = mode == 0 && fa.unit_volume && first_small_pencils(p, p.metric, &PB);
    a.PB = PB;
    a.d_PB = FastDiv::make((uint32_t)PB);
    a.nbd = FastDiv::make((uint32_t)(PB * DIM));
    a.nblk = (int)((a.inner_total + PB - 1) / PB);
    if (fa.partial && (size_t)a.nblk > p.part_stride)
        return set_error(FEH_EINVAL, "first axis: more partial sums than a row of them holds");
    const bool table = mode == 0 && fa.unit_volume;
    const bool perlc = table ? first_by_table(p, p.metric) : first_per_load_case(p);
    a.total = perlc ? a.nblk * p.L : a.nblk;  // one block per (load case, pencils) or per pencils
    dim3 g(a.total), b(kFftThreads);
    const size_t tab_dyn = ((a.n0 * sizeof(Cx<T>) + 15) / 16) * 16 + (mode == 0 ? 4 * (size_t)PB * sizeof(Cx<double>) : 0);
    if ((small ? ppt<T, true>() : PPT) * kFftThreads * sizeof(Cx<T>) + (kFftThreads / 64) * sizeof(double) + tab_dyn > kLdsPerWorkgroup)
        return set_error(FEH_ENOTSUP, "first axis too long for the LDS transform");
    // general lengths: a tile of the pass's own size, 16 bytes a multiple (see
    // lds_of_pass); with the largest tile one FP64 workgroup of 1661 points
    // had a CU to itself (1661^2 by strains, a solve: 19.7 -> 16.7 ms)
    constexpr int kAlign = 16 / (int)sizeof(Cx<T>);
    a.lbuf = pow2_len(a.n0) ? 0 : (a.n0 * PB * DIM + kAlign - 1) / kAlign * kAlign;
    const size_t dyn = (size_t)a.lbuf * sizeof(Cx<T>) + tab_dyn;
    // the CG's fused pass (element volume relative to the voxel) reads the
    // (B^*B)^-1 table, built here on the first use for this workspace and
    // block size; the test exports (true volume) form the inverses in place
    const bool tab = table && perlc;
    if (tab) {
        a.minv = p.ptr<T>(p.off_minv);
        // the compile-time pass reads the table with lane-interleaved slots
        a.minv_q = ctpb > 0 ? 16 / (int)sizeof(T) : 0;
        const int rc = ensure_table<T, DIM>(p, a);
        if (rc != FEH_OK) return rc;
    }
    if (ctpb > 0) {
        switch (a.n0) {
        case 64: hipLaunchKernelGGL((k_first_ct<T, 64, DIM>), g, b, 0, p.stream, a); break;
        case 128: hipLaunchKernelGGL((k_first_ct<T, 128, DIM>), g, b, 0, p.stream, a); break;
        case 256: hipLaunchKernelGGL((k_first_ct<T, 256, DIM>), g, b, 0, p.stream, a); break;
        case 1024:
            if constexpr (sizeof(T) == 4 || DIM == 2) hipLaunchKernelGGL((k_first_ct<T, 1024, DIM>), g, b, 0, p.stream, a);
            break;
        default: hipLaunchKernelGGL((k_first_ct<T, 512, DIM>), g, b, 0, p.stream, a); break;
        }
        return hip_check(hipGetLastError(), "first-axis fft launch");
    }
    auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, g, b, dyn, p.stream, a); };
    with_gen(a.ax, [&](auto gl) {
        constexpr int G = decltype(gl)::value;
        auto layouts = [&](auto m) {
            constexpr int M = decltype(m)::value;
            if (perlc) run(k_first<T, PPT, DIM, M, G, true, false>);
            else run(k_first<T, PPT, DIM, M, G, false, false>);
        };
        if (small) run(k_first<T, ppt<T, true>(), DIM, 0, G, true, true>);
        else if (tab) run(k_first<T, PPT, DIM, 0, G, true, true>);
        else if (mode == 0) layouts(std::integral_constant<int, 0>{});
        else if (mode == 1) layouts(std::integral_constant<int, 1>{});
        else layouts(std::integral_constant<int, 2>{});
    });
    return hip_check(hipGetLastError(), "first-axis fft launch");
}

template <typename T>
int first_dispatch(const feh_plan &p, const FftArgs &fa, int mode) {
    return p.dim == 3 ? first_t<T, 3>(p, fa, mode) : first_t<T, 2>(p, fa, mode);
}

}  // namespace

// Default first-axis layout of the passes that form their inverses: one
// workgroup per (load case, pencil block) when the axis length is a power of
// two.  That variant forms the inverses again per load case but fits 3 waves
// per SIMD (FP32; 2 in FP64, bound by LDS) against 2 (FP32) or 1 (FP64) for
// the register-cached variant, and runs faster at every measured size.
// General lengths keep the cached variant (both hold about as many registers
// there).
bool first_per_load_case(const feh_plan &p) {
    if (p.tune_first_perlc != 0) return p.tune_first_perlc > 0;
    return pow2_len((int)p.n[0]);
}

// Pencils per block of the compile-time first-axis pass of the CG, or 0 when
// the plan's shape or schedule has none: a power-of-two axis 0 of 64 to 1024
// points (1024: FP64 in 2D only) in the default radix order, the default layout (one workgroup
// per load case) and block size, and offsets that fit the 24-bit products
// of the staging.
int first_ct_pencils(const feh_plan &p) {
    const int n0 = (int)p.n[0];
    if (!p.tune_ct || p.tune_pb_first != 0 || !first_per_load_case(p)) return 0;
    // 1024 points: two pencils, at most half a CU's LDS.  The run-time pass's
    // tile and twiddles took just more than half of it in FP64, so that each of
    // its workgroups had a CU to itself (1024^2 x 3 load cases: a pass 78 us,
    // a solve 27.6 -> 22.7 ms)
    const bool two = n0 == 1024 && (p.prec == FEH_FP32 || p.dim == 2);
    if (!(n0 == 64 || n0 == 128 || n0 == 256 || n0 == 512 || two) || !ct_schedule_matches(p.fft[0], n0)) return 0;
    const long long inner = p.dim == 3 ? p.n[1] * p.nh : p.nh;
    const long long rowD = inner * p.dim;
    if (rowD >= (1 << 24) || rowD * n0 >= (1ll << 31)) return 0;
    return two ? 2 : (p.prec == FEH_FP32 ? 2048 : 1024) / n0;
}

// The CG's first-axis pass reads its inverses from the table, one workgroup
// per load case: where the schedule has that layout, for every metric other
// than 0 (the table is the only place of its inverses), and at every length
// that is not a power of two, whose layout 0 is thus one of the passes that
// form their inverses only.  The table pass has n_load times the workgroups of
// the cached variant at no arithmetic more.  A solve of 24 iterations, cached
// and by table, FP32: 45 x 50 x 39 x 6 load cases 1.69 and 0.94 ms, 160^3 x 6
// 15.4 and 13.1, 300^2 x 3 1.25 and 0.62, 900^2 x 1 1.04 and 0.99; FP64:
// 151^2 x 3 5.49 and 1.64, 900^2 x 1 2.65 and 2.65, 90 x 77 x 105 x 6 19.3 and
// 16.1.  Of 48 such solves one was slower, 1661 x 300 x 1 in FP32 (1.22 and
// 1.26 ms).
bool first_by_table(const feh_plan &p, int metric) {
    return first_per_load_case(p) || metric != 0 || !pow2_len((int)p.n[0]);
}

int first_pencils_default(const feh_plan &p) {
    const int PPT = p.prec == FEH_FP32 ? 24 : 16;
    int PB = (PPT * kFftThreads) / (int)(p.n[0] * p.dim);
    if (PB < 1) PB = 1;
    if (PB > 32) PB = 32;
    return PB;
}

int first_num_parts(const feh_plan &p) { return first_num_parts(p, p.metric); }

int first_num_parts(const feh_plan &p, int metric) {
    int PB = first_pencils_default(p);
    // tuned value, never below a quarter of the default: the partial-sum
    // buffer holds one slot per pencil block for that size
    if (p.tune_pb_first > 0 && p.tune_pb_first < PB) PB = std::max(p.tune_pb_first, std::max(1, PB / 4));
    if (const int ct = first_ct_pencils(p)) PB = ct;  // the CG's fused pass
    const long long inner = p.dim == 3 ? p.n[1] * p.nh : p.nh;
    if (PB > inner) PB = (int)inner;
    (void)first_small_pencils(p, metric, &PB);
    return (int)((inner + PB - 1) / PB);
}

int launch_inverse_table(const feh_plan &p) {
    if (p.prec == FEH_FP64) return p.dim == 3 ? plain_table<double, 3>(p) : plain_table<double, 2>(p);
    return p.dim == 3 ? plain_table<float, 3>(p) : plain_table<float, 2>(p);
}

int launch_forward_last(const feh_plan &p, const FftArgs &a) {
    return p.prec == FEH_FP64 ? last_t<double>(p, a, false) : last_t<float>(p, a, false);
}
int launch_inverse_last(const feh_plan &p, const FftArgs &a) {
    return p.prec == FEH_FP64 ? last_t<double>(p, a, true) : last_t<float>(p, a, true);
}
int launch_middle(const feh_plan &p, const FftArgs &a, bool inverse) {
    return p.prec == FEH_FP64 ? middle_t<double>(p, a, inverse) : middle_t<float>(p, a, inverse);
}
int launch_first_fused(const feh_plan &p, const FftArgs &a) {
    return p.prec == FEH_FP64 ? first_dispatch<double>(p, a, 0) : first_dispatch<float>(p, a, 0);
}
int launch_first_plain(const feh_plan &p, const FftArgs &a, bool inverse) {
    return p.prec == FEH_FP64 ? first_plain_t<double>(p, a, inverse) : first_plain_t<float>(p, a, inverse);
}
int launch_first(const feh_plan &p, const FftArgs &a, bool inverse) {
    const int mode = inverse ? 2 : 1;
    return p.prec == FEH_FP64 ? first_dispatch<double>(p, a, mode) : first_dispatch<float>(p, a, mode);
}

}  // namespace feh
