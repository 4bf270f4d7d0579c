// fp64_math.hpp -- lean float64 exp and softplus for the bound search (device and host).
//
//  exp(x):  Cody-Waite reduction x = k ln2 + r, |r| <= ln2 / 2 (ln2 split into a 53-bit head and
//           its remainder), exp(r) by its Taylor polynomial of degree 13 (truncation < 5e-18
//           relative on that range), scaled by 2^k.  For |x| <= 700.
//  log1p(t) for 0 <= t <= 1:  log(1 + t) = 2 atanh(u), u = t / (2 + t) in [0, 1/3], by the odd
//           series 2 (u + u^3/3 + u^5/5 + ...) to u^35 (truncation < 1e-17 relative).
//  softplus(x) = log(1 + e^x) = max(x, 0) + log1p(e^-|x|).
//
// For the Phase II/III posterior, whose time is its float64 operations, the same functions from
// Chebyshev expansions of the same accuracy and fewer terms (computed with 60 digits, then written in
// powers), and the complementary error function:
//  exp_short:    degree 11 on |r| <= ln2 / 2 (3e-18 relative; Taylor needs 13);
//  log1p_short:  atanh(u) / u in u^2 on [0, 1/9], degree 10 (1.3e-18; the odd series needs 17);
//  erfc_pos(x), x >= 0: (1 + 2x) exp(x^2) erfc(x) in t = (x - 3.75) / (x + 3.75) on [0, 27], degree 24
//                (5e-19; the variable and the factor are Shepherd and Laframboise's, Math. Comp. 36
//                (1981) 249), times exp(-x^2) with x^2 in two parts; error below 7e-16 relative, no
//                branches (the library's takes up to 170 float64 operations, this one 60).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>

namespace cse {

__host__ __device__ __forceinline__ double exp_cw(double x) {
    const double ln2_hi = 0x1.62e42fefa39efp-1;    // nearest double to ln 2
    const double ln2_lo = 0x1.abc9e3b39803fp-56;   // ln 2 - ln2_hi
    const double k = rint(x * 0x1.71547652b82fep0);  // x / ln 2
    const double r = fma(-k, ln2_lo, fma(-k, ln2_hi, x));
    double p = 1.0 / 6227020800.0;   // 1/13!
    p = fma(p, r, 1.0 / 479001600.0);
    p = fma(p, r, 1.0 / 39916800.0);
    p = fma(p, r, 1.0 / 3628800.0);
    p = fma(p, r, 1.0 / 362880.0);
    p = fma(p, r, 1.0 / 40320.0);
    p = fma(p, r, 1.0 / 5040.0);
    p = fma(p, r, 1.0 / 720.0);
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return ldexp(p, (int)k);
}

// log(1 + t) = 2 atanh(u) from u = t / (2 + t) in [0, 1/3].
__host__ __device__ __forceinline__ double log1p_from_u(double u) {
    const double w = u * u;
    double s = 1.0 / 35.0;
#pragma unroll
    for (int j = 33; j >= 1; j -= 2) s = fma(s, w, 1.0 / (double)j);
    return 2.0 * u * s;
}

__host__ __device__ __forceinline__ double log1p_unit(double t) { return log1p_from_u(t / (2.0 + t)); }

__host__ __device__ __forceinline__ double softplus_fast(double x) {
    return fmax(x, 0.0) + log1p_unit(exp_cw(-fabs(x)));
}

__host__ __device__ __forceinline__ double exp_short(double x) {
    const double ln2_hi = 0x1.62e42fefa39efp-1;
    const double ln2_lo = 0x1.abc9e3b39803fp-56;
    const double k = rint(x * 0x1.71547652b82fep0);
    const double r = fma(-k, ln2_lo, fma(-k, ln2_hi, x));
    double p = 0x1.af785e0a5dff9p-26;
    p = fma(p, r, 0x1.28b40639f7187p-22);
    p = fma(p, r, 0x1.71dde76a2f6d2p-19);
    p = fma(p, r, 0x1.a01991aba6f13p-16);
    p = fma(p, r, 0x1.a01a01b802660p-13);
    p = fma(p, r, 0x1.6c16c187fc3e6p-10);
    p = fma(p, r, 0x1.111111110db75p-7);
    p = fma(p, r, 0x1.555555554f0ccp-5);
    p = fma(p, r, 0x1.5555555555562p-3);
    p = fma(p, r, 0x1.0000000000011p-1);
    p = fma(p, r, 0x1.0000000000000p+0);
    p = fma(p, r, 0x1.0000000000000p+0);
    return ldexp(p, (int)k);
}

// log(1 + t) from u = t / (2 + t) in [0, 1/3].
__host__ __device__ __forceinline__ double log1p_short(double u) {
    const double w = u * u;
    double p = 0x1.5d5192c5c16ebp-4;
    p = fma(p, w, 0x1.54b093b32599bp-5);
    p = fma(p, w, 0x1.f01958209fc71p-5);
    p = fma(p, w, 0x1.10632786a2475p-4);
    p = fma(p, w, 0x1.3b1e423307d9fp-4);
    p = fma(p, w, 0x1.745cae5cdec88p-4);
    p = fma(p, w, 0x1.c71c744e01706p-4);
    p = fma(p, w, 0x1.2492492009c9cp-3);
    p = fma(p, w, 0x1.99999999a1ed1p-3);
    p = fma(p, w, 0x1.5555555555526p-2);
    p = fma(p, w, 0x1.0000000000000p+0);
    return 2.0 * u * p;
}

// erfc(x), x >= 0 (26.5 at most: erfc(26.5) = 1e-307 is returned beyond), given 1/d by `rcp`.
template <class Rcp>
__host__ __device__ __forceinline__ double erfc_pos(double x, Rcp rcp) {
    x = fmin(x, 26.5);
    const double xk = x + 3.75, x2 = fma(2.0, x, 1.0);
    const double inv = rcp(xk * x2);
    const double t = (x - 3.75) * x2 * inv;
    double p = 0x1.3ca2ccf44e0eap-32;
    p = fma(p, t, -0x1.21acc9eca0446p-33);
    p = fma(p, t, -0x1.62ff4043b4f1dp-28);
    p = fma(p, t, -0x1.455830fc6d8fep-29);
    p = fma(p, t, 0x1.53d4826b32fc9p-25);
    p = fma(p, t, 0x1.70bf79080a7e3p-26);
    p = fma(p, t, -0x1.17a96df5a1870p-22);
    p = fma(p, t, -0x1.e0ae19471cc9bp-25);
    p = fma(p, t, 0x1.d6aa84805a019p-20);
    p = fma(p, t, -0x1.0577de51656e8p-20);
    p = fma(p, t, -0x1.800909b09078cp-17);
    p = fma(p, t, 0x1.778becdfdc1e5p-16);
    p = fma(p, t, 0x1.b14461532c864p-15);
    p = fma(p, t, -0x1.303fa3fc51fe8p-12);
    p = fma(p, t, 0x1.33fb23804e4f0p-12);
    p = fma(p, t, 0x1.cc3a0e5ed7c79p-10);
    p = fma(p, t, -0x1.3f603c3295dfbp-7);
    p = fma(p, t, 0x1.d0b0037d73c6bp-6);
    p = fma(p, t, -0x1.e0d0fa6e066e5p-5);
    p = fma(p, t, 0x1.7a14188a9ad76p-4);
    p = fma(p, t, -0x1.bda9309a286ddp-4);
    p = fma(p, t, 0x1.510169d096792p-4);
    p = fma(p, t, 0x1.d5f2948159c58p-9);
    p = fma(p, t, -0x1.1f367683f89a6p-3);
    p = fma(p, t, 0x1.3ccda0b5d5dc2p+0);
    const double h = x * x, l = fma(x, x, -h);
    const double e = exp_short(-h);
    return p * (xk * inv) * fma(-e, l, e);
}

}  // namespace cse
