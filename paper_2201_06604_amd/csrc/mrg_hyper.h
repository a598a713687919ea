// mrg_hyper.h -- one contingency-table entry by inversion of its conditional
// hypergeometric distribution (Section 4), host and device.
//
// Definition (the one the oracle evaluates, hyper_invert): x in [lo, hi] with
// weights w(lo) = 1, w(x+1) = w(x) * ((K-x)(n-x)) / ((x+1)(N'-K-n+x+1)) in
// double precision (exact integer products, one rounded multiply, one rounded
// divide); the entry is the smallest x with u*W <= w(lo)+...+w(x), sums
// ascending.  Weights above 2^600 and the running sum are scaled by 2^-600
// (exact), and the search compares u*W with the running sum at W's scale:
// the mantissas of the same operations on an unbounded exponent range.
//
// hyper_search gives the same x from one pass over part of the range, with no
// division in its loop and bounds on all roundings, or says that the bounds do
// not decide; then the definition does.
#pragma once

#include <stdint.h>

#include <cmath>

#ifndef MRG_HD
#if defined(__HIPCC__)
#define MRG_HD __host__ __device__
#else
#define MRG_HD
#endif
#endif

namespace mrg355 {

constexpr double kHyperBig = 0x1p600;
constexpr int kHyperScaleExp = 600;

// The definition.  The integer products of the ratio are formed in fp64: with
// every total at most 2^20 (the callers' bound) each factor is an integer
// below 2^21 and each product below 2^42, so the fp64 products are exact and
// equal the integer products converted to double.  The first pass (W) stops
// once the ratio has dropped below 1 (the weights only decrease from there:
// num/den <= 1 - 2^-40, so even after two roundings each weight is below the
// previous one) and the next weight is below W * 2^-54 (under half an ulp of
// W): every later addition rounds back to W.
MRG_HD inline int hyper_invert(double u, int Np, int K, int n) {
    const int lo = n - (Np - K) > 0 ? n - (Np - K) : 0;
    const int hi = n < K ? n : K;
    if (hi <= lo) return lo;
    const double Kd = K, nd = n, rest = Np - K - n + 1;  // N' - K - n + 1
    double W = 0.0, w = 1.0, xd = lo;
    int scales = 0;
    for (int x = lo; x <= hi; ++x, xd += 1.0) {
        W += w;
        if (x < hi) {
            const double num = (Kd - xd) * (nd - xd);
            const double den = (xd + 1.0) * (rest + xd);
            w = w * num / den;
            if (w > kHyperBig) {
                w = ldexp(w, -kHyperScaleExp);
                W = ldexp(W, -kHyperScaleExp);
                ++scales;
            }
            if (num < den && w * 0x1p54 < W) break;
        }
    }
    const double target = u * W;
    double s = 0.0;
    w = 1.0;
    xd = lo;
    int done = 0;
    for (int x = lo; x <= hi; ++x, xd += 1.0) {
        s += w;
        if (target <= ldexp(s, -kHyperScaleExp * (scales - done))) return x;
        const double num = (Kd - xd) * (nd - xd);
        const double den = (xd + 1.0) * (rest + xd);
        w = w * num / den;
        if (w > kHyperBig) {
            w = ldexp(w, -kHyperScaleExp);
            s = ldexp(s, -kHyperScaleExp);
            ++done;
        }
    }
    return hi;
}

// 1/x to about 2^-22, for choices that need no more.
MRG_HD inline float hyper_rcp(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_rcpf(x);
#else
    return 1.0f / x;
#endif
}

MRG_HD inline float hyper_sqrt(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_sqrtf(x);
#else
    return sqrtf(x);
#endif
}

// The same x, or -1 where the bounds below do not decide it.  lf(k) is
// log(k!) rounded to double, 0 <= k <= N' <= 2^20; lfN = lf(N') on entry and
// lf(N' - K) on return (the next entry's).
//
// The whole W is a binomial coefficient, so in units of the weight at any x0
// the target u*W is T = u / pmf(x0), by log-factorials.  x0 lies `reach`
// standard deviations and two below the mean (or at lo): the weights below it
// sum to at most tau = rho / (1 - rho), rho the ratio of the first of them to
// w(x0), since the ratios only get smaller downwards.  From x0 the running sum
// is carried as a quotient A/D with w(x) = N/D, and the target as V = T D:
//   V <- V den(x),  N <- N num(x),  A <- A den(x) + N,
// three operations and no division a step; num and den, second-order
// polynomials in x, step by their differences, exactly.  Four steps run between
// comparisons; the first x with A >= V is then found by taking weights off A.
//
// What separates this from the definition, relative to u*W (eps = 2^-53):
// the definition's own roundings, at most 6 (hi - lo) + 1 eps (two a weight and
// one a sum, on both sides of the comparison); those of A and V, at most
// 3 (hi - lo) + 4 eps; and those of T: the nine logarithms sum to at most
// 4 log(N'!) in magnitude, so their table errors and eight additions are within
// 36 log(N'!) eps, exp and the product within 8 eps.  gam bounds the sum with
// room for the few roundings of the last comparisons, all relative to the
// largest A, and tau/T is added below.  The answer is given where the sums up
// to x and to x - 1 differ from the target by more than that; u falls nearer
// than that to a step of the distribution function in about 1e-9 of all draws at
// N' = 12,900 and 1e-7 at 2^20, and near or below the first attempt's x0 in about 1e-5.
//
// A shorter first reach saves steps and sends more lanes (and with them their
// whole wave) round again: the paper's month test took 3.19 / 2.39 / 2.34 / 2.42
// ms at 3.5 / 4 / 4.5 / 5, 10^6 small tables 205 / 203 / 209 / 213 us.
constexpr float kHyperNear = 4.25f, kHyperFar = 9.0f;  // reach of the two attempts
constexpr int kHyperBlock = 4;
constexpr int kHyperRescale = 4;  // blocks: 16 products below 2^42 and T < 2^100 stay below 2^772

template <typename LogFact>
MRG_HD inline int hyper_search(double u, int Np, int K, int n, double& lfN, LogFact lf) {
    const int lo = n - (Np - K) > 0 ? n - (Np - K) : 0;
    const int hi = n < K ? n : K;
    const double lf_rest = lf(Np - K);
    const double lf_whole = lfN;
    lfN = lf_rest;
    if (hi <= lo) return lo;
    const double lf_fixed = (lf(K) + lf_rest) + ((lf(n) + lf(Np - n)) - lf_whole);
    const double gam = 0x1p-53 * (48.0 * (lf_whole + 8.0) + 16.0 * (hi - lo));
    // any x0 in [lo, hi) will do: single precision
    const float inv = hyper_rcp(static_cast<float>(Np));
    const float share = static_cast<float>(K) * inv;
    const float mean = static_cast<float>(n) * share;
    const float dev = hyper_sqrt(mean * (1.0f - share) * (static_cast<float>(Np - n) * inv));
    float reach = kHyperNear;
    for (;;) {
        int x0 = static_cast<int>(mean - reach * dev) - 2;
        if (x0 > hi - 1) x0 = hi - 1;
        if (x0 < lo) x0 = lo;
        // log pmf(x0), and T = u / pmf(x0)
        const double y = lf_fixed - ((lf(x0) + lf(K - x0)) + (lf(n - x0) + lf(Np - K - n + x0)));
        const double T = u * exp(-y);
        const double a = K - x0, b = n - x0, c = x0, d = Np - K - n + x0;
        double num = a * b, dnum = 1.0 - a - b;                    // num(x+1) = num(x) + dnum, dnum + 2 next
        double den = (c + 1.0) * (d + 1.0), dden = c + d + 3.0;  // den(x+1) = den(x) + dden, dden + 2 next
        double below = 0.0;  // tau
        bool fair = T < 0x1p100;
        if (x0 > lo) {
            const double first = c * d, one = num + (a + b) + 1.0;  // rho = first / one, one = (a + 1)(b + 1)
            fair = fair && first < one;
            below = static_cast<double>(static_cast<float>(first) * hyper_rcp(static_cast<float>(one - first)) * 1.01f);
        }
        if (fair) {
            double A = 1.0, V = T, N = 1.0;
            double N1 = 0.0, N2 = 0.0, N3 = 0.0, d2 = 1.0, d3 = 1.0, d4 = 1.0;
            int x = x0;
            // Past hi (num was 0 there, so N is 0 from then on) A/V no longer
            // changes: a lane may run on to the end of its block.
            for (int block = 0; A < V && x < hi; x += kHyperBlock) {
                V *= den;
                N1 = N * num;
                A = __builtin_fma(A, den, N1);
                num += dnum; dnum += 2.0; den += dden; dden += 2.0;
                d2 = den;
                V *= d2;
                N2 = N1 * num;
                A = __builtin_fma(A, d2, N2);
                num += dnum; dnum += 2.0; den += dden; dden += 2.0;
                d3 = den;
                V *= d3;
                N3 = N2 * num;
                A = __builtin_fma(A, d3, N3);
                num += dnum; dnum += 2.0; den += dden; dden += 2.0;
                d4 = den;
                V *= d4;
                N = N3 * num;
                A = __builtin_fma(A, d4, N);
                num += dnum; dnum += 2.0; den += dden; dden += 2.0;
                if (++block == kHyperRescale && A < V) {
                    block = 0;
                    int e;
                    frexp(V, &e);
                    A = ldexp(A, -e);
                    V = ldexp(V, -e);
                    N = ldexp(N, -e);
                }
            }
            if (A >= V) {
                // A holds the sum up to x; top and S become those up to the first
                // x with top >= V and up to x - 1
                const double room = (gam + static_cast<double>(hyper_rcp(static_cast<float>(T))) * below) * A;
                double top = A, S = A - N;
                if (x > x0) {
                    double back = d4;
                    if (S >= V) {
                        top = S; --x; S = top - N3 * back; back *= d3;
                        if (S >= V) {
                            top = S; --x; S = top - N2 * back; back *= d2;
                            if (S >= V) { top = S; --x; S = top - N1 * back; }
                        }
                    }
                }
                // past x = hi - 1 the definition stops at hi, whatever the sum
                if (S <= V - room && (x == hi || top >= V + room)) return x;
            }
        }
        if (reach == kHyperFar) return -1;
        reach = kHyperFar;
    }
}

}  // namespace mrg355
