// md.hpp -- device multiple-double arithmetic for gfx950.
//
// An m-double is M binary64 limbs, limb 0 most significant, denoting the
// exact sum of its limbs.  The operations follow the project's fixed
// specification (error-free transformations, level sums, renormalisation);
// they are fully unrolled at compile time, branch-free and data-independent,
// so a wavefront never diverges inside an operation.  Build with
// -ffp-contract=off and without fast-math: every + - * below is one IEEE
// round-to-nearest operation and __builtin_fma is the fused one.
//
//   two_sum(a, b)   s = a+b, e = (a-(s-bb)) + (b-bb), bb = s-a   (Knuth)
//   two_prod(a, b)  p = a*b, e = fma(a, b, -p)
//   deposit<LO>     add t into the level sums S[LO..M-1]; exact until the
//                   last level, which adds plainly
//   renorm          bottom-up two_sum pass, then top-down two_sum pass
//   md_add(x, y)    S = x; deposit y_k at level k; renorm
//   md_mul(x, y)    exact products of levels 0..M-2, plain FMAs for levels
//                   M-1 and M, exact low parts pushed one level down; renorm
//
// Complex m-doubles (real and imaginary parts kept apart, Sections 2 and 5)
// are 2M doubles, the real limbs then the imaginary ones:
//   cmd_mul(x, y)   re = md_add(xr*yr, -(xi*yi)), im = md_add(xr*yi, xi*yr),
//                   each product an md_mul, the negation exact
//   cmd_add(x, y)   md_add of the real parts and of the imaginary parts
#pragma once

#include <hip/hip_runtime.h>

// At the top of a kernel: counts the last accumulation register as used (no
// instruction), so that a wavefront holds more than half of its SIMD's 512
// registers and no two of them share a SIMD.  For launches of one-wavefront
// workgroups that fill a SIMD once at most: the dispatcher's placement goes on
// from the launch before, and without this it puts two of them on one SIMD
// beside an idle one or not, whichever way the earlier workgroups fell (a last
// layer of 910 of p1's: eight doubles and d = 95 2800 or 3091 us the whole
// evaluation, ten and d = 31 751 or 874).  Four wavefronts per workgroup spread
// as evenly, but slow a lone wavefront of ten doubles (d = 64: 1158 -> 1232 us).
__device__ __forceinline__ void one_per_simd() { asm volatile("" ::: "a255"); }

#include <type_traits>

namespace mdpe {

template <int B, int E, class F>
__device__ __forceinline__ void sfor(F &&f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        sfor<B + 1, E>(f);
    }
}

// R doubles of R independent coefficients, worked on element by element.  A
// multiple-double operation on Vec<R> issues every step for all R before the
// next one, so a dependent FP64 instruction follows R - 1 independent ones: a
// lone wavefront then no longer waits out each result's latency (a dependent
// FP64 addition can issue about two issue slots after its operand).
template <int R>
struct Vec {
    double v[R];
};

#define MDPE_VEC_OP(op)                                                                   \
    template <int R>                                                                      \
    __device__ __forceinline__ Vec<R> operator op(const Vec<R> &a, const Vec<R> &b) {     \
        Vec<R> c;                                                                         \
        _Pragma("unroll") for (int r = 0; r < R; ++r) c.v[r] = a.v[r] op b.v[r];          \
        return c;                                                                         \
    }
MDPE_VEC_OP(+)
MDPE_VEC_OP(-)
MDPE_VEC_OP(*)
#undef MDPE_VEC_OP

template <int R>
__device__ __forceinline__ Vec<R> operator*(double a, const Vec<R> &b) {
    Vec<R> c;
#pragma unroll
    for (int r = 0; r < R; ++r) c.v[r] = a * b.v[r];
    return c;
}
template <int R>
__device__ __forceinline__ Vec<R> operator*(const Vec<R> &a, double b) {
    Vec<R> c;
#pragma unroll
    for (int r = 0; r < R; ++r) c.v[r] = a.v[r] * b;
    return c;
}
template <int R>
__device__ __forceinline__ Vec<R> operator-(const Vec<R> &a) {
    Vec<R> c;
#pragma unroll
    for (int r = 0; r < R; ++r) c.v[r] = -a.v[r];
    return c;
}

__device__ __forceinline__ double md_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }
template <int R>
__device__ __forceinline__ Vec<R> md_fma(double a, const Vec<R> &b, const Vec<R> &c) {
    Vec<R> z;
#pragma unroll
    for (int r = 0; r < R; ++r) z.v[r] = __builtin_fma(a, b.v[r], c.v[r]);
    return z;
}
template <int R>
__device__ __forceinline__ Vec<R> md_fma(const Vec<R> &a, double b, const Vec<R> &c) {
    Vec<R> z;
#pragma unroll
    for (int r = 0; r < R; ++r) z.v[r] = __builtin_fma(a.v[r], b, c.v[r]);
    return z;
}

// Every operation below is written once for T = double and T = Vec<R>; the
// factors X and Y of a product may be one double (shared by the R
// coefficients) or a Vec.
template <class T>
__device__ __forceinline__ void two_sum(T a, T b, T &s, T &e) {
    T ss = a + b;
    T bb = ss - a;
    e = (a - (ss - bb)) + (b - bb);
    s = ss;
}

template <class X, class Y, class T>
__device__ __forceinline__ void two_prod(X a, Y b, T &p, T &e) {
    T pp = a * b;
    e = md_fma(a, b, -pp);
    p = pp;
}

template <int M, int LO, class T>
__device__ __forceinline__ void deposit(T (&S)[M], T t) {
    if constexpr (LO < M - 1) {
        two_sum(S[LO], t, S[LO], t);
        deposit<M, LO + 1>(S, t);
    } else {
        S[M - 1] = S[M - 1] + t;
    }
}

template <int M, class T>
__device__ __forceinline__ void renorm(const T (&S)[M], T (&r)[M]) {
    if constexpr (M == 1) {
        r[0] = S[0];
    } else {
        T u[M];
        T s = S[M - 1];
        sfor<0, M - 1>([&](auto q) {
            constexpr int j = M - 2 - decltype(q)::value;
            two_sum(S[j], s, s, u[j + 1]);
        });
        u[0] = s;
        r[0] = u[0];
        T e = u[1];
        sfor<1, M - 1>([&](auto q) {
            constexpr int j = decltype(q)::value;
            two_sum(e, u[j + 1], r[j], e);
        });
        r[M - 1] = e;
    }
}

template <int M, class T>
__device__ __forceinline__ void md_add(const T (&x)[M], const T (&y)[M], T (&z)[M]) {
    T S[M];
    sfor<0, M>([&](auto k) { S[decltype(k)::value] = x[decltype(k)::value]; });
    sfor<0, M>([&](auto k) {
        constexpr int K = decltype(k)::value;
        deposit<M, K>(S, y[K]);
    });
    renorm<M>(S, z);
}

template <int M, class X, class Y, class T>
__device__ __forceinline__ void md_mul(const X (&x)[M], const Y (&y)[M], T (&z)[M]) {
    T S[M];
    T E[M > 1 ? M - 1 : 1];
    sfor<0, M - 1>([&](auto k) {
        constexpr int K = decltype(k)::value;
        two_prod(x[0], y[K], S[K], E[K]);
    });
    S[M - 1] = x[0] * y[M - 1];
    sfor<1, M>([&](auto i) {
        constexpr int I = decltype(i)::value;
        S[M - 1] = md_fma(x[I], y[M - 1 - I], S[M - 1]);
    });
    sfor<1, M>([&](auto i) {
        constexpr int I = decltype(i)::value;
        S[M - 1] = md_fma(x[I], y[M - I], S[M - 1]);
    });
    sfor<0, M - 1>([&](auto k) {
        constexpr int K = decltype(k)::value;
        deposit<M, K + 1>(S, E[K]);
    });
    sfor<1, M - 1>([&](auto k) {
        constexpr int K = decltype(k)::value;
        sfor<1, K + 1>([&](auto i) {
            constexpr int I = decltype(i)::value;
            T p, e;
            two_prod(x[I], y[K - I], p, e);
            deposit<M, K>(S, p);
            deposit<M, K + 1>(S, e);
        });
    });
    renorm<M>(S, z);
}

// Doubles per coefficient: M limbs, or 2M for complex series.
template <int M, bool CX>
constexpr int kCoef = CX ? 2 * M : M;

template <int M, class X, class Y, class T>
__device__ __forceinline__ void cmd_mul(const X (&x)[2 * M], const Y (&y)[2 * M], T (&z)[2 * M]) {
    X xr[M], xi[M];
    Y yr[M], yi[M];
    sfor<0, M>([&](auto l) {
        constexpr int L = decltype(l)::value;
        xr[L] = x[L];
        xi[L] = x[M + L];
        yr[L] = y[L];
        yi[L] = y[M + L];
    });
    T rr[M], ii[M], ri[M], ir[M], zr[M], zi[M];
    md_mul<M>(xr, yr, rr);
    md_mul<M>(xi, yi, ii);
    md_mul<M>(xr, yi, ri);
    md_mul<M>(xi, yr, ir);
    sfor<0, M>([&](auto l) { ii[decltype(l)::value] = -ii[decltype(l)::value]; });
    md_add<M>(rr, ii, zr);
    md_add<M>(ri, ir, zi);
    sfor<0, M>([&](auto l) {
        constexpr int L = decltype(l)::value;
        z[L] = zr[L];
        z[M + L] = zi[L];
    });
}

template <int M, class T>
__device__ __forceinline__ void cmd_add(const T (&x)[2 * M], const T (&y)[2 * M], T (&z)[2 * M]) {
    T xr[M], xi[M], yr[M], yi[M], zr[M], zi[M];
    sfor<0, M>([&](auto l) {
        constexpr int L = decltype(l)::value;
        xr[L] = x[L];
        xi[L] = x[M + L];
        yr[L] = y[L];
        yi[L] = y[M + L];
    });
    md_add<M>(xr, yr, zr);
    md_add<M>(xi, yi, zi);
    sfor<0, M>([&](auto l) {
        constexpr int L = decltype(l)::value;
        z[L] = zr[L];
        z[M + L] = zi[L];
    });
}

// One coefficient operation of the series' number field.
template <int M, bool CX, class X, class Y, class T>
__device__ __forceinline__ void coef_mul(const X (&x)[kCoef<M, CX>], const Y (&y)[kCoef<M, CX>],
                                         T (&z)[kCoef<M, CX>]) {
    if constexpr (CX)
        cmd_mul<M>(x, y, z);
    else
        md_mul<M>(x, y, z);
}

template <int M, bool CX, class T>
__device__ __forceinline__ void coef_add(const T (&x)[kCoef<M, CX>], const T (&y)[kCoef<M, CX>],
                                         T (&z)[kCoef<M, CX>]) {
    if constexpr (CX)
        cmd_add<M>(x, y, z);
    else
        md_add<M>(x, y, z);
}

}  // namespace mdpe
