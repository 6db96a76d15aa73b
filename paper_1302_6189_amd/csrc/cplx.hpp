// cplx.hpp -- complex arithmetic and small DFT butterflies for the FFT passes.
//
// Every butterfly computes y_k = sum_j w^{jk} x_j for a short length R, the
// 1-D DFT of Eq. (1), with w = exp(DIR * 2 pi i / R): DIR = -1 is the paper's
// forward transform, DIR = +1 the (unscaled) inverse.  The formulas are the
// usual splittings of that sum into even/odd or symmetric parts.
//
// Every product that is added to something is written as a fused
// multiply-add, so no contraction is left to the compiler: the same
// butterflies give the same bits in every kernel they are inlined in (the
// fused and the separate kernels of a step are compared bit for bit).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace fftrw {

template <typename Real> struct CplxOf;
template <> struct CplxOf<float> { using type = float2; };
template <> struct CplxOf<double> { using type = double2; };

template <typename C> struct RealOf;
template <> struct RealOf<float2> { using type = float; };
template <> struct RealOf<double2> { using type = double; };

// Pointers that a kernel reads out of a descriptor in memory are generic
// (flat) pointers to the compiler, and flat accesses count on the LDS wait
// counter as well: a wait for one LDS read then also waits for every flat
// load and store still in flight, which serialises a thread's HBM accesses.
// Passing such a pointer through the global address space lets the compiler
// issue global_ loads and stores, whose waits are separate from the LDS's.
template <typename T> __device__ __forceinline__ T *as_global(T *p)
{
    return (T *)(__attribute__((address_space(1))) T *)p;
}

// HBM accesses through the global address space.  A pointer a kernel reads
// out of a descriptor in memory is a generic (flat) pointer to the compiler,
// and flat accesses count on the LDS wait counter too: a wait for one LDS
// read then also waits for every flat load and store still in flight, which
// serialises a thread's HBM accesses.  Global loads and stores have waits of
// their own.  Only for pointers into device memory (never LDS).
template <typename T> __device__ __forceinline__ T gld_nt(const T *p)
{
    return __builtin_nontemporal_load((const __attribute__((address_space(1))) T *)p);
}
template <typename T> __device__ __forceinline__ void gst_nt(T v, T *p)
{
    __builtin_nontemporal_store(v, (__attribute__((address_space(1))) T *)p);
}
template <typename T> __device__ __forceinline__ void gst(T v, T *p) { *(__attribute__((address_space(1))) T *)p = v; }
// Calls f(std::true_type()) or f(std::false_type()) by a uniform choice of
// streaming or cached accesses.  Of two branches that differ in the kind of
// their accesses alone the compiler makes one, cached; the empty statements
// that differ from branch to branch keep them apart.
template <typename F> __device__ __forceinline__ void either(bool nt, F &&f)
{
    if (nt) {
        asm volatile("; streaming" ::: "memory");
        f(std::true_type());
        asm volatile("; streaming done" ::: "memory");
    } else {
        asm volatile("; cached" ::: "memory");
        f(std::false_type());
        asm volatile("; cached done" ::: "memory");
    }
}
// one complex value (float2 or double2), cached
template <typename T> __device__ __forceinline__ T gld(const T *p)
{
    if constexpr (sizeof(T) == 8) {
        typedef float v2 __attribute__((ext_vector_type(2)));
        const v2 w = *(const __attribute__((address_space(1))) v2 *)p;
        T r;
        r.x = w.x;
        r.y = w.y;
        return r;
    } else {
        typedef double v2 __attribute__((ext_vector_type(2)));
        const v2 w = *(const __attribute__((address_space(1))) v2 *)p;
        T r;
        r.x = w.x;
        r.y = w.y;
        return r;
    }
}

template <typename C> __device__ __forceinline__ C mk(typename RealOf<C>::type x, typename RealOf<C>::type y)
{
    C r;
    r.x = x;
    r.y = y;
    return r;
}
template <typename C> __device__ __forceinline__ C cadd(C a, C b) { return mk<C>(a.x + b.x, a.y + b.y); }
template <typename C> __device__ __forceinline__ C csub(C a, C b) { return mk<C>(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
template <typename C> __device__ __forceinline__ C cmul(C a, C b)
{
    return mk<C>(fma_(a.x, b.x, -(a.y * b.y)), fma_(a.x, b.y, a.y * b.x));
}
// a * conj(b)
template <typename C> __device__ __forceinline__ C cmulc(C a, C b)
{
    return mk<C>(fma_(a.x, b.x, a.y * b.y), fma_(a.y, b.x, -(a.x * b.y)));
}
// c + s a
template <typename C> __device__ __forceinline__ C cfma(typename RealOf<C>::type s, C a, C c)
{
    return mk<C>(fma_(s, a.x, c.x), fma_(s, a.y, c.y));
}
template <typename C> __device__ __forceinline__ C cscale(C a, typename RealOf<C>::type s)
{
    return mk<C>(a.x * s, a.y * s);
}
// a * (DIR * i)
template <int DIR, typename C> __device__ __forceinline__ C rot90(C a)
{
    return DIR < 0 ? mk<C>(a.y, -a.x) : mk<C>(-a.y, a.x);
}
// twiddle product: a * w (forward) or a * conj(w) (inverse); w from a forward table
template <int DIR, typename C> __device__ __forceinline__ C twmul(C a, C w)
{
    return DIR < 0 ? cmul(a, w) : cmulc(a, w);
}

// a * (x + i y) for a constant of a butterfly.  In single precision the constant
// enters in two parts: its rounding would be in every output that it reaches,
// in pass after pass (complex64 rows of 2187 points, radix 9, err by 1.36e-7
// with rounded constants, 1.29e-7 with two parts and 1.32e-7 in radix 3; 4096
// points, radix 16, by 1.21e-7, 1.17e-7 and, in radix 8, 1.19e-7).
template <typename C> __device__ __forceinline__ C cmulk(C a, double x, double y)
{
    if constexpr (sizeof(C) == 8) {
        const float hx = (float)x, hy = (float)y, lx = (float)(x - (double)hx), ly = (float)(y - (double)hy);
        const C e = cmul(a, mk<C>(lx, ly));
        return mk<C>(fma_(a.x, hx, fma_(-a.y, hy, e.x)), fma_(a.x, hy, fma_(a.y, hx, e.y)));
    } else {
        return cmul(a, mk<C>(x, y));
    }
}

template <int R, int DIR, typename C> struct Dft;

template <int DIR, typename C> struct Dft<2, DIR, C> {
    static __device__ __forceinline__ void run(C *x)
    {
        C a = x[0], b = x[1];
        x[0] = cadd(a, b);
        x[1] = csub(a, b);
    }
};

template <int DIR, typename C> struct Dft<4, DIR, C> {
    static __device__ __forceinline__ void run(C *x)
    {
        C a = cadd(x[0], x[2]), b = csub(x[0], x[2]);
        C c = cadd(x[1], x[3]), d = rot90<DIR>(csub(x[1], x[3]));
        x[0] = cadd(a, c);
        x[2] = csub(a, c);
        x[1] = cadd(b, d);
        x[3] = csub(b, d);
    }
};

template <int DIR, typename C> struct Dft<8, DIR, C> {
    static __device__ __forceinline__ void run(C *x)
    {
        using Real = typename RealOf<C>::type;
        const Real h = (Real)0.70710678118654752440084436210485;
        C e[4] = {x[0], x[2], x[4], x[6]};
        C o[4] = {x[1], x[3], x[5], x[7]};
        Dft<4, DIR, C>::run(e);
        Dft<4, DIR, C>::run(o);
        // w8^k = (cos(pi k/4), DIR sin(pi k/4)): odd k are h times a sum or
        // difference of the parts, added with one fma each
        C o1 = mk<C>(o[1].x - DIR * o[1].y, o[1].y + DIR * o[1].x);
        C o2 = rot90<DIR>(o[2]);
        C o3 = mk<C>(-o[3].x - DIR * o[3].y, -o[3].y + DIR * o[3].x);
        x[0] = cadd(e[0], o[0]);
        x[4] = csub(e[0], o[0]);
        x[1] = cfma(h, o1, e[1]);
        x[5] = cfma(-h, o1, e[1]);
        x[2] = cadd(e[2], o2);
        x[6] = csub(e[2], o2);
        x[3] = cfma(h, o3, e[3]);
        x[7] = cfma(-h, o3, e[3]);
    }
};

// 4 x 4: column DFTs, twiddles w16^{i k}, row DFTs
template <int DIR, typename C> struct Dft<16, DIR, C> {
    static __device__ __forceinline__ void run(C *x)
    {
        using Real = typename RealOf<C>::type;
        const Real h = (Real)0.70710678118654752440084436210485;
        const double c1 = 0.92387953251128675612818318939679;  // cos(pi/8)
        const double s1 = 0.38268343236508977172845998403040;  // sin(pi/8)
        C c[4][4];  // c[n][k]: column n (inputs n + 4 i), output k
#pragma unroll
        for (int n = 0; n < 4; ++n) {
#pragma unroll
            for (int i = 0; i < 4; ++i) c[n][i] = x[n + 4 * i];
            Dft<4, DIR, C>::run(c[n]);
        }
        // terms that w16^2 = h (1 + DIR i) or w16^6 = h (-1 + DIR i) multiplies
        // keep the factor h for the fma that adds them
        const C t12 = mk<C>(c[1][2].x - DIR * c[1][2].y, c[1][2].y + DIR * c[1][2].x);
        const C t21 = mk<C>(c[2][1].x - DIR * c[2][1].y, c[2][1].y + DIR * c[2][1].x);
        const C t23 = mk<C>(-c[2][3].x - DIR * c[2][3].y, -c[2][3].y + DIR * c[2][3].x);
        const C t32 = mk<C>(-c[3][2].x - DIR * c[3][2].y, -c[3][2].y + DIR * c[3][2].x);
        // row 0: no twiddles
        C r0[4] = {c[0][0], c[1][0], c[2][0], c[3][0]};
        Dft<4, DIR, C>::run(r0);
        // rows 1 and 3: column 2 enters times h
        auto odd = [&](C z0, C z1, C t2, C z3, int k) {
            const C a = cfma(h, t2, z0), b = cfma(-h, t2, z0);
            const C c_ = cadd(z1, z3), d = rot90<DIR>(csub(z1, z3));
            x[k] = cadd(a, c_);
            x[k + 8] = csub(a, c_);
            x[k + 4] = cadd(b, d);
            x[k + 12] = csub(b, d);
        };
        odd(c[0][1], cmulk(c[1][1], c1, DIR * s1), t21, cmulk(c[3][1], s1, DIR * c1), 1);
        odd(c[0][3], cmulk(c[1][3], s1, DIR * c1), t23, cmulk(c[3][3], -c1, -DIR * s1), 3);
        // row 2: columns 1 and 3 enter times h, column 2 times DIR i
        {
            const C z2 = rot90<DIR>(c[2][2]);
            const C a = cadd(c[0][2], z2), b = csub(c[0][2], z2);
            const C p = cadd(t12, t32), q = rot90<DIR>(csub(t12, t32));
            x[2] = cfma(h, p, a);
            x[10] = cfma(-h, p, a);
            x[6] = cfma(h, q, b);
            x[14] = cfma(-h, q, b);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) x[4 * i] = r0[i];
    }
};

template <int DIR, typename C> struct Dft<3, DIR, C> {
    static __device__ __forceinline__ void run(C *x)
    {
        using Real = typename RealOf<C>::type;
        const Real s3 = (Real)0.86602540378443864676372317075294;
        C t = cadd(x[1], x[2]);
        C m = cfma((Real)-0.5, t, x[0]);
        C s = rot90<DIR>(csub(x[1], x[2]));
        x[0] = cadd(x[0], t);
        x[1] = cfma(s3, s, m);
        x[2] = cfma(-s3, s, m);
    }
};

// The sines enter each output on their own: sin(2 pi/5) (b1 + q b2) with the
// ratio q of the two sines has two operations less, but both roundings in
// every output, and complex64 rows of 625 and 3125 points then err by 1.33
// and 1.51e-7 instead of 1.21 and 1.35e-7 (against 80 bits).
template <int DIR, typename C> struct Dft<5, DIR, C> {
    static __device__ __forceinline__ void run(C *x)
    {
        using Real = typename RealOf<C>::type;
        const Real c1 = (Real)0.30901699437494742410229341718282;   // cos(2 pi/5)
        const Real c2 = (Real)-0.80901699437494742410229341718282;  // cos(4 pi/5)
        const Real s1 = (Real)0.95105651629515357211643933337938;   // sin(2 pi/5)
        const Real s2 = (Real)0.58778525229247312916870595463907;   // sin(4 pi/5)
        C a1 = cadd(x[1], x[4]), a2 = cadd(x[2], x[3]);
        C b1 = rot90<DIR>(csub(x[1], x[4])), b2 = rot90<DIR>(csub(x[2], x[3]));
        C y0 = cadd(x[0], cadd(a1, a2));
        C m1 = cfma(c2, a2, cfma(c1, a1, x[0]));
        C m2 = cfma(c1, a2, cfma(c2, a1, x[0]));
        x[0] = y0;
        x[1] = cfma(s1, b1, cfma(s2, b2, m1));
        x[4] = cfma(-s1, b1, cfma(-s2, b2, m1));
        x[2] = cfma(-s1, b2, cfma(s2, b1, m2));
        x[3] = cfma(s1, b2, cfma(-s2, b1, m2));
    }
};

// Length A B with coprime A and B (Good 1958): input (B a + A b) mod A B and
// output k with k = ka mod A, k = kb mod B turn the sum into an A x B DFT with
// no twiddles in between.
template <int A, int B, int DIR, typename C> struct DftCoprime {
    static constexpr int out(int ka, int kb)
    {
        int k = ka;
        while (k % B != kb) k += A;
        return k;
    }
    static __device__ __forceinline__ void run(C *x)
    {
        C t[A][B];
#pragma unroll
        for (int a = 0; a < A; ++a) {
#pragma unroll
            for (int b = 0; b < B; ++b) t[a][b] = x[(B * a + A * b) % (A * B)];
            Dft<B, DIR, C>::run(t[a]);
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            C r[A];
#pragma unroll
            for (int a = 0; a < A; ++a) r[a] = t[a][b];
            Dft<A, DIR, C>::run(r);
#pragma unroll
            for (int a = 0; a < A; ++a) x[out(a, b)] = r[a];
        }
    }
};
template <int DIR, typename C> struct Dft<6, DIR, C> : DftCoprime<2, 3, DIR, C> {};
template <int DIR, typename C> struct Dft<10, DIR, C> : DftCoprime<2, 5, DIR, C> {};
template <int DIR, typename C> struct Dft<12, DIR, C> : DftCoprime<4, 3, DIR, C> {};
template <int DIR, typename C> struct Dft<15, DIR, C> : DftCoprime<3, 5, DIR, C> {};

// 3 x 3: column DFTs, twiddles w9^{i k}, row DFTs
template <int DIR, typename C> struct Dft<9, DIR, C> {
    static __device__ __forceinline__ void run(C *x)
    {
        C c[3][3];
#pragma unroll
        for (int n = 0; n < 3; ++n) {
#pragma unroll
            for (int i = 0; i < 3; ++i) c[n][i] = x[n + 3 * i];
            Dft<3, DIR, C>::run(c[n]);
        }
        // w9^1, w9^2, w9^2 and w9^4
        c[1][1] = cmulk(c[1][1], 0.76604444311897803520239265055542, DIR * 0.64278760968653932632264340990726);
        c[1][2] = cmulk(c[1][2], 0.17364817766693034885171662676931, DIR * 0.98480775301220805936674302458952);
        c[2][1] = cmulk(c[2][1], 0.17364817766693034885171662676931, DIR * 0.98480775301220805936674302458952);
        c[2][2] = cmulk(c[2][2], -0.93969262078590838405410927732473, DIR * 0.34202014332566873304409961468226);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            C r[3] = {c[0][k], c[1][k], c[2][k]};
            Dft<3, DIR, C>::run(r);
#pragma unroll
            for (int i = 0; i < 3; ++i) x[k + 3 * i] = r[i];
        }
    }
};

// exp(-2 pi i e / n), 0 <= e < n <= 2^28: the angle is reduced to an octant in
// integers, so that its rounding is a share of an angle of at most pi / 4
// (-2 e / n rounded as it is puts up to several units of the last place into
// the roots of every n that is no power of two: complex128 rows of 320 points
// 2.34e-16 instead of 2.19e-16, of 81 points 2.19e-16 instead of 1.96e-16).
__device__ inline void unit_root(int e, int n, double *re, double *im)
{
    const int o = 8 * e / n, r = 8 * e - o * n;
    double s, c;
    sincospi((double)(o % 2 ? n - r : r) / (4.0 * (double)n), &s, &c);
    double x = o % 2 ? s : c, y = o % 2 ? c : s;
    const int q = o / 2;  // quarter turns
    if (q % 2) {
        const double t = x;
        x = -y;
        y = t;
    }
    *re = q >= 2 ? -x : x;
    *im = q >= 2 ? y : -y;
}

}  // namespace fftrw
