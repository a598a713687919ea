// The bounded entry search against the definition it stands for, on the host:
//   hyper_search_xcheck CASES MAX_TOTAL SEED STEPS
// CASES random entries (all kinds of margins, uniforms next to 0, to 1 and at simple
// fractions among them) and STEPS entries at uniforms on both sides of a step of the
// distribution function, found by bisection.  The search may leave an entry to the
// definition (-1) but never give another.  Prints cases, undecided ones and wrong ones.
#include <math.h>

#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "mrg_hyper.h"

using namespace mrg355;

int main(int argc, char** argv) {
    if (argc != 5) return 2;
    const long cases = atol(argv[1]), steps = atol(argv[4]);
    const int max_total = atoi(argv[2]);
    std::mt19937_64 g(static_cast<unsigned long>(atol(argv[3])));
    std::vector<double> lf(static_cast<size_t>(max_total) + 1);
    for (size_t k = 0; k < lf.size(); ++k) {
        int sign;
        lf[k] = static_cast<double>(lgammal_r(static_cast<long double>(k) + 1.0L, &sign));
    }
    const auto logfact = [&](int k) {
        if (k < 0 || k > max_total) abort();
        return lf[static_cast<size_t>(k)];
    };
    long undecided = 0, wrong = 0, seen = 0;
    const auto check = [&](double u, int Np, int K, int n) {
        double lfN = logfact(Np);
        const int got = hyper_search(u, Np, K, n, lfN, logfact);
        ++seen;
        if (lfN != logfact(Np - K)) ++wrong;
        if (got < 0) {
            ++undecided;
        } else if (got != hyper_invert(u, Np, K, n)) {
            if (wrong++ < 5) printf("N=%d K=%d n=%d u=%.17g: %d\n", Np, K, n, u, got);
        }
    };
    const auto margins = [&](int& Np, int& K, int& n) {
        Np = 1 + static_cast<int>(exp(std::uniform_real_distribution<double>(0.0, log(max_total - 1.0))(g)));
        switch (g() % 4) {
            case 0: K = g() % (Np + 1); n = g() % (Np + 1); break;
            case 1: K = g() % (Np / 10 + 1); n = g() % (Np / 10 + 1); break;
            case 2: K = Np - g() % (Np / 20 + 1); n = g() % (Np + 1); break;
            default: K = g() % (Np < 30 ? Np + 1 : 30); n = Np - g() % (Np < 40 ? Np + 1 : 40);
        }
    };
    int Np, K, n;
    for (long i = 0; i < cases; ++i) {
        margins(Np, K, n);
        uint64_t z = 1 + g() % 4294967087ull;  // MRG32k3a's uniforms are z / 4294967088
        switch (g() % 4) {
            case 0: z = 1 + g() % 8; break;
            case 1: z = 4294967087ull - g() % 8; break;
            case 2: z = (1 + g() % 15) * 268435443ull; break;
        }
        check(static_cast<double>(z) * (1.0 / 4294967088.0), Np, K, n);
    }
    for (long i = 0; i < steps; ++i) {
        margins(Np, K, n);
        double below = std::uniform_real_distribution<double>(0x1p-33, 1.0)(g), above = 1.0 - 0x1p-53;
        const int x = hyper_invert(below, Np, K, n);
        if (hyper_invert(above, Np, K, n) == x) continue;
        while (nextafter(below, 1.0) < above) {
            const double mid = below + 0.5 * (above - below);
            (hyper_invert(mid, Np, K, n) == x ? below : above) = mid;
        }
        for (int k = 0; k < 60; k += 4) {  // from the step itself to a relative 2^-4 off it
            check(below * (1.0 - ldexp(1.0, k - 60)), Np, K, n);
            check(fmin(above * (1.0 + ldexp(1.0, k - 60)), 1.0 - 0x1p-53), Np, K, n);
        }
    }
    printf("%ld cases, %ld undecided, %ld wrong\n", seen, undecided, wrong);
    return wrong != 0;
}
