// Butterflies of the transforms on registers, and the matrix-core tile of the
// prime passes.  Shared by the passes of kern_fft.hip and kern_small.hip
// (internal linkage).
#pragma once

#include "device_common.hpp"

namespace feh {
namespace {

template <typename T>
__device__ __forceinline__ Cx<T> mul_mi(Cx<T> a) { return {a.y, -a.x}; }  // a * (-i)
template <typename T>
__device__ __forceinline__ Cx<T> mul_pi(Cx<T> a) { return {-a.y, a.x}; }  // a * (+i)
template <typename T>
__device__ __forceinline__ Cx<T> cscale(Cx<T> a, T s) { return {a.x * s, a.y * s}; }

template <typename T>
__device__ __forceinline__ Cx<T> twid(const Cx<T> *tw, int tws, int e, bool inv) {
    Cx<T> w = tw[e * tws];
    if (inv) w.y = -w.y;
    return w;
}

// In-place DFT of length R on registers: x[d] <- sum_c x[c] exp(-+2 pi i c d / R).
template <typename T, int R>
struct Dft {
    // generic radix (7, 11, 13): roots from the table of the full length n
    static __device__ __forceinline__ void run(Cx<T> (&x)[R], bool inv, const Cx<T> *tw, int tws, int n) {
        Cx<T> y[R];
        const int step = n / R;
        #pragma unroll
        for (int d = 0; d < R; ++d) {
            Cx<T> s = x[0];
            #pragma unroll
            for (int c = 1; c < R; ++c) s = cadd(s, cmul(x[c], twid(tw, tws, ((c * d) % R) * step, inv)));
            y[d] = s;
        }
        #pragma unroll
        for (int d = 0; d < R; ++d) x[d] = y[d];
    }
};

template <typename T>
struct Dft<T, 2> {
    static __device__ __forceinline__ void run(Cx<T> (&x)[2], bool, const Cx<T> *, int, int) {
        const Cx<T> a = x[0];
        x[0] = cadd(a, x[1]);
        x[1] = csub(a, x[1]);
    }
};

template <typename T>
struct Dft<T, 3> {
    static __device__ __forceinline__ void run(Cx<T> (&x)[3], bool inv, const Cx<T> *, int, int) {
        const T s3 = T(0.86602540378443864676);
        const Cx<T> t1 = cadd(x[1], x[2]), t2 = csub(x[1], x[2]);
        const Cx<T> a = {x[0].x - T(0.5) * t1.x, x[0].y - T(0.5) * t1.y};
        const Cx<T> b = cscale(t2, s3);
        x[0] = cadd(x[0], t1);
        if (!inv) {
            x[1] = cadd(a, mul_mi(b));
            x[2] = cadd(a, mul_pi(b));
        } else {
            x[1] = cadd(a, mul_pi(b));
            x[2] = cadd(a, mul_mi(b));
        }
    }
};

template <typename T>
__device__ __forceinline__ void dft4(Cx<T> &x0, Cx<T> &x1, Cx<T> &x2, Cx<T> &x3, bool inv) {
    const Cx<T> a = cadd(x0, x2), b = csub(x0, x2), c = cadd(x1, x3), d = csub(x1, x3);
    x0 = cadd(a, c);
    x2 = csub(a, c);
    if (!inv) {
        x1 = cadd(b, mul_mi(d));
        x3 = cadd(b, mul_pi(d));
    } else {
        x1 = cadd(b, mul_pi(d));
        x3 = cadd(b, mul_mi(d));
    }
}

template <typename T>
struct Dft<T, 4> {
    static __device__ __forceinline__ void run(Cx<T> (&x)[4], bool inv, const Cx<T> *, int, int) {
        dft4(x[0], x[1], x[2], x[3], inv);
    }
};

template <typename T>
struct Dft<T, 5> {
    static __device__ __forceinline__ void run(Cx<T> (&x)[5], bool inv, const Cx<T> *, int, int) {
        const T c1 = T(0.30901699437494742410), c2 = T(-0.80901699437494742410);
        const T s1 = T(0.95105651629515357212), s2 = T(0.58778525229247312917);
        const Cx<T> t1 = cadd(x[1], x[4]), t2 = cadd(x[2], x[3]);
        const Cx<T> t3 = csub(x[1], x[4]), t4 = csub(x[2], x[3]);
        const Cx<T> a1 = {x[0].x + c1 * t1.x + c2 * t2.x, x[0].y + c1 * t1.y + c2 * t2.y};
        const Cx<T> a2 = {x[0].x + c2 * t1.x + c1 * t2.x, x[0].y + c2 * t1.y + c1 * t2.y};
        const Cx<T> b1 = {s1 * t3.x + s2 * t4.x, s1 * t3.y + s2 * t4.y};
        const Cx<T> b2 = {s2 * t3.x - s1 * t4.x, s2 * t3.y - s1 * t4.y};
        x[0] = cadd(x[0], cadd(t1, t2));
        if (!inv) {
            x[1] = cadd(a1, mul_mi(b1));
            x[4] = cadd(a1, mul_pi(b1));
            x[2] = cadd(a2, mul_mi(b2));
            x[3] = cadd(a2, mul_pi(b2));
        } else {
            x[1] = cadd(a1, mul_pi(b1));
            x[4] = cadd(a1, mul_mi(b1));
            x[2] = cadd(a2, mul_pi(b2));
            x[3] = cadd(a2, mul_mi(b2));
        }
    }
};

template <typename T>
struct Dft<T, 8> {
    static __device__ __forceinline__ void run(Cx<T> (&x)[8], bool inv, const Cx<T> *, int, int) {
        const T h = T(0.70710678118654752440);
        Cx<T> e0 = x[0], e1 = x[2], e2 = x[4], e3 = x[6];
        Cx<T> o0 = x[1], o1 = x[3], o2 = x[5], o3 = x[7];
        dft4(e0, e1, e2, e3, inv);
        dft4(o0, o1, o2, o3, inv);
        // o_d *= W8^d, W8 = exp(-+ i pi / 4)
        if (!inv) {
            o1 = {h * (o1.x + o1.y), h * (o1.y - o1.x)};
            o2 = mul_mi(o2);
            o3 = {h * (o3.y - o3.x), -h * (o3.x + o3.y)};
        } else {
            o1 = {h * (o1.x - o1.y), h * (o1.x + o1.y)};
            o2 = mul_pi(o2);
            o3 = {-h * (o3.x + o3.y), h * (o3.x - o3.y)};
        }
        x[0] = cadd(e0, o0);
        x[4] = csub(e0, o0);
        x[1] = cadd(e1, o1);
        x[5] = csub(e1, o1);
        x[2] = cadd(e2, o2);
        x[6] = csub(e2, o2);
        x[3] = cadd(e3, o3);
        x[7] = csub(e3, o3);
    }
};

// Matrix-core tile D = A B + C of 16 rows, 16 columns and 4 inner steps (one
// wavefront): lane l holds A(l % 16, l / 16) and B(l / 16, l % 16).
template <typename T>
struct Mfma;
template <>
struct Mfma<double> {
    typedef double Acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ Acc run(double a, double b, Acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * r + (lane >> 4); }  // of c[r]
};
template <>
struct Mfma<float> {
    typedef float Acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ Acc run(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

}  // namespace
}  // namespace feh
