// mrg_engine.h -- the exact generator steps on gfx950 (device code, included
// by the kernel sources).  MRG32k3a in two interchangeable arithmetic forms:
//
//   IntEngine    32x32->64 multiply-adds, reduced with 2^32 = c (mod 2^32 - c)
//   F64EngineOf  the same integers held exactly in fp64: every product is below
//                2^53 and each remainder p - q*m is one exact FMA
//
// Both give identical integers z in [1, m1].  MRG31k3p runs in the fp64 form
// only.
//
// Every engine keeps each component as a ring of three registers holding
// (x[n-3], x[n-2], x[n-1]); a step overwrites x[n-3] with x[n], so a 3-step
// cycle needs no register moves.  Both recurrences read x1[n-2], x1[n-3],
// x2[n-1] and x2[n-3], so the ring logic is shared.
#pragma once

#include <hip/hip_runtime.h>

#include "mrg_logtab.h"
#include "mrg_sincostab.h"
#include "mrg_math.h"

namespace mrg355 {

// -------------------------------------------------------- integer engine
// p < 2^54 -> p mod m1.  p = h*2^32 + l with h < 2^22; 2^32 = 209 (mod m1).
__device__ __forceinline__ uint32_t fold_m1(uint64_t p) {
    uint32_t h = static_cast<uint32_t>(p >> 32), l = static_cast<uint32_t>(p);
    uint64_t t = static_cast<uint64_t>(__umul24(h, kC1)) + l;          // < 2^32 + 2^30
    uint32_t r = static_cast<uint32_t>(t) + static_cast<uint32_t>(t >> 32) * kC1;
    return min(r, r - kM1);                                             // r < 2^32 < 2 m1
}

// p < 2^54 -> p mod m2.  h < 2^21, 2^32 = 22853 (mod m2).
__device__ __forceinline__ uint32_t fold_m2(uint64_t p) {
    uint32_t h = static_cast<uint32_t>(p >> 32), l = static_cast<uint32_t>(p);
    uint64_t t = static_cast<uint64_t>(h) * kC2 + l;                   // < 2^36 + 2^32
    uint32_t h2 = static_cast<uint32_t>(t >> 32), l2 = static_cast<uint32_t>(t);
    uint64_t t2 = static_cast<uint64_t>(__umul24(h2, kC2)) + l2;       // < 2^32 + 2^19
    uint32_t r = static_cast<uint32_t>(t2) + static_cast<uint32_t>(t2 >> 32) * kC2;
    return min(r, r - kM2);
}

struct IntEngine {
    struct Regs {};  // its constants are literals
    uint32_t a0, a1, a2, b0, b1, b2;  // (x1[n-3], x1[n-2], x1[n-1]), (x2[...])

    __device__ __forceinline__ void load(const uint32_t x[6]) {
        a0 = x[0]; a1 = x[1]; a2 = x[2]; b0 = x[3]; b1 = x[4]; b2 = x[5];
    }
    __device__ __forceinline__ void save(uint32_t x[6]) const {
        x[0] = a0; x[1] = a1; x[2] = a2; x[3] = b0; x[4] = b1; x[5] = b2;
    }
    // New x1 from (x1[n-2], x1[n-3]) replaces x1[n-3]; new x2 from (x2[n-1],
    // x2[n-3]) replaces x2[n-3]; returns z in [1, m1].
    static __device__ __forceinline__ uint32_t kernel(uint32_t& o1, uint32_t m2_1, uint32_t& o2,
                                                      uint32_t n1_2) {
        uint64_t p1 = static_cast<uint64_t>(kA12) * m2_1 + static_cast<uint64_t>(kA13N) * (kM1 - o1);
        uint64_t p2 = static_cast<uint64_t>(kA21) * n1_2 + static_cast<uint64_t>(kA23N) * (kM2 - o2);
        uint32_t x1 = fold_m1(p1), x2 = fold_m2(p2);
        o1 = x1;
        o2 = x2;
        return x1 > x2 ? x1 - x2 : x1 - x2 + kM1;
    }
    // Phase-P step of a 3-step cycle: the ring of registers rotates by naming,
    // so no moves are needed.
    template <int P>
    __device__ __forceinline__ uint32_t step(const Regs&) {
        if (P == 0) return kernel(a0, a1, b0, b2);
        if (P == 1) return kernel(a1, a2, b1, b0);
        return kernel(a2, a0, b2, b1);
    }
    __device__ __forceinline__ uint32_t step_rot(const Regs&) {
        uint32_t z = kernel(a0, a1, b0, b2);
        uint32_t t = a0; a0 = a1; a1 = a2; a2 = t;
        t = b0; b0 = b1; b1 = b2; b2 = t;
        return z;
    }
};

// ------------------------------------------------------------ fp64 engine
// Constants of generator G in fp64.  Both components are carried less half of
// the second modulus, h = (m2 - 1)/2, so a recurrence
//   x[n] = (p x[n-i] + q x[n-3]) mod m   becomes   c[n] = p c[n-i] + q c[n-3] + K (mod m)
// on c = x - h with K = (p + q - 1) h mod m, the representative nearest zero.
template <int G>
struct F64Consts {
    static constexpr bool k32 = G == kGen32k3a;
    static constexpr uint32_t m1w = k32 ? kM1 : kP1, m2w = k32 ? kM2 : kP2;
    static constexpr int64_t p1w = k32 ? kA12 : kB12, q1w = k32 ? -static_cast<int64_t>(kA13N) : kB13;
    static constexpr int64_t p2w = k32 ? kA21 : kB21, q2w = k32 ? -static_cast<int64_t>(kA23N) : kB23;
    static constexpr uint32_t hw = (m2w - 1) / 2;
    static constexpr double m1 = m1w, h = hw;
    static constexpr double centred(int64_t x, int64_t m) {
        x %= m;
        if (2 * x > m) x -= m;
        if (2 * x < -m) x += m;
        return static_cast<double>(x);
    }
};

// The constants of a step, held in registers.  The empty asm hides their
// values: with literals the compiler turns the multiply-adds into the
// accumulating form, which overwrites its addend, and copies every addend
// first (115 VALU instructions per six fp64 uniforms instead of 84).  Made
// once, before the loops.
template <int G>
struct F64Regs {
    using C = F64Consts<G>;
    double p1, q1, K1, p2, q2, K2, m1, m2, inv1, inv2;
    double shift;   // 1.5 2^52: adding it rounds to an integer
    double shift_v; // the same in vector registers (an instruction reads one scalar pair)
    __device__ __forceinline__ F64Regs()
        : p1(C::p1w), q1(C::q1w), K1(C::centred((C::p1w + C::q1w - 1) * C::hw, C::m1w)), p2(C::p2w), q2(C::q2w),
          K2(C::centred((C::p2w + C::q2w - 1) * C::hw, C::m2w)), m1(C::m1w), m2(C::m2w), inv1(1.0 / C::m1w),
          inv2(1.0 / C::m2w), shift(0x1.8p52), shift_v(0x1.8p52) {
        asm("" : "+s"(p1), "+s"(q1), "+s"(p2), "+s"(q2), "+s"(m1), "+s"(m2), "+s"(inv1), "+s"(inv2), "+s"(shift));
        asm("" : "+v"(K1), "+v"(K2), "+v"(shift_v));
    }
};

// p an integer, |p| <= (p1 + |q1|) (m/2 + 2^14) + m/2 < 2^53 -> an integer
// r = p (mod m) with |r| <= m/2 + 1, exactly.  The quotient is one FMA onto
// 1.5 2^52, whose last place is 1, so it is p/m rounded once, with the
// error of the constant 1/m alone before the rounding; p - q*m is exact.
//
// Where |p| < 0.906 2^20 m the result is the residue in [-(m-1)/2, (m-1)/2]:
// p/m is at least 1/(2m) > 2^-33 away from any half integer (m is odd) and
// the constant's error moves it by at most 2^-53 |p/m| < 2^-33.14.
template <int G>
__device__ __forceinline__ double f64_centred(double p, double m, double inv_m, const F64Regs<G>& k) {
    const double q = __builtin_fma(p, inv_m, k.shift_v) - k.shift;
    return __builtin_fma(-q, m, p);
}

// 1 where the integer d is 0 or less, 0 where it is 1 or more: 1 - d clamped
// to [0, 1], one instruction.
__device__ __forceinline__ double f64_wraps(double d) {
    return __builtin_fmin(__builtin_fmax(1.0 - d, 0.0), 1.0);
}

// One step of a component costs two multiply-adds, the quotient's two
// instructions and the remainder's one; z costs three more: 13 per integer,
// 14 per fp64 uniform (17 and 18 with component 2 kept in [0, m2) by a floor
// step and z found by another: 2^28 f32 uniforms of 65,536 streams 203 -> 179
// us, 2^30 fp64 normals 1844 -> 1771 us; MRG31k3p took about 30 as 32-bit
// rotations and folds, and its 10^8 normals of the paper's example 225 -> 205
// us).  Issue-bound: every instruction here takes one slot.
//
// Component 1 may be any residue with |a| <= m1/2 + 1 (its class mod m1 is
// what matters).  Component 2 must be one value per class, because z uses it:
// its |p| is at most (p2 + |q2| + 1) m2/2 < 0.906 2^20 m2, so f64_centred
// gives the residue in [-h, h], and x2 = b + h lies in [0, m2).  A state just
// loaded has a in [-h, m1 - h), a few thousand past m1/2, which the bound on p
// allows for.
template <int G>
struct F64EngineOf {
    using C = F64Consts<G>;
    using Regs = F64Regs<G>;
    double a0, a1, a2, b0, b1, b2;  // (x1[n-3], x1[n-2], x1[n-1]) - h, (x2[...]) - h

    __device__ __forceinline__ void load(const uint32_t x[6]) {
        // MRG31k3p's stored state is newest first
        a0 = x[C::k32 ? 0 : 2] - C::h; a1 = x[1] - C::h; a2 = x[C::k32 ? 2 : 0] - C::h;
        b0 = x[C::k32 ? 3 : 5] - C::h; b1 = x[4] - C::h; b2 = x[C::k32 ? 5 : 3] - C::h;
    }
    static __device__ __forceinline__ uint32_t word1(double a) {  // a + h is below m1: add m1 where negative
        const double v = a + C::h;
        return static_cast<uint32_t>(__builtin_fma(f64_wraps(v + 1.0), C::m1, v));
    }
    __device__ __forceinline__ void save(uint32_t x[6]) const {
        x[C::k32 ? 0 : 2] = word1(a0);
        x[1] = word1(a1);
        x[C::k32 ? 2 : 0] = word1(a2);
        x[C::k32 ? 3 : 5] = static_cast<uint32_t>(b0 + C::h);
        x[4] = static_cast<uint32_t>(b1 + C::h);
        x[C::k32 ? 5 : 3] = static_cast<uint32_t>(b2 + C::h);
    }
    // o1 = c1[n-3] (becomes c1[n]), m2_1 = c1[n-2], o2 = c2[n-3] (becomes
    // c2[n]), n1_2 = c2[n-1]; returns z in [1, m1].
    static __device__ __forceinline__ double kernel(const Regs& k, double& o1, double m2_1, double& o2, double n1_2) {
        const double t1 = __builtin_fma(k.q1, o1, k.K1);
        const double t2 = __builtin_fma(k.q2, o2, k.K2);
        o1 = f64_centred<G>(__builtin_fma(k.p1, m2_1, t1), k.m1, k.inv1, k);
        o2 = f64_centred<G>(__builtin_fma(k.p2, n1_2, t2), k.m2, k.inv2, k);
        // h cancels: d = x1 - x2 (mod m1) with |d| <= (m1 + m2)/2 + 1 < m1
        const double d = o1 - o2;
        return __builtin_fma(f64_wraps(d), k.m1, d);
    }
    template <int P>
    __device__ __forceinline__ double step(const Regs& k) {
        if (P == 0) return kernel(k, a0, a1, b0, b2);
        if (P == 1) return kernel(k, a1, a2, b1, b0);
        return kernel(k, a2, a0, b2, b1);
    }
    __device__ __forceinline__ double step_rot(const Regs& k) {
        double z = kernel(k, a0, a1, b0, b2);
        double t = a0; a0 = a1; a1 = a2; a2 = t;
        t = b0; b0 = b1; b1 = b2; b2 = t;
        return z;
    }
};

// ------------------------------------------------------------- transforms
// sqrt(x) for the Box-Muller radius argument x = -2 log(u1) in [2^-32, 47]:
// never zero, subnormal or non-finite, so the range scaling and special
// cases of a general square root are left out.  Goldschmidt's iteration from
// the hardware reciprocal square root y ~ 1/sqrt(x): g ~ sqrt(x) and
// h ~ 1/(2 sqrt(x)) are refined together once, then one Newton correction
// g += h (x - g^2) with an exact residual (FMA).  mrg_transform_accuracy
// compares it with the HIP library's sqrt on the radius argument of any range
// of generator outputs: bit-identical over every output of both generators
// (a second correction changed no result).
__device__ __forceinline__ double sqrt_radius(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y;
    double h = 0.5 * y;
    const double r = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, r, g);
    h = __builtin_fma(h, r, h);
    const double d = __builtin_fma(-g, g, x);
    return __builtin_fma(d, h, g);
}

// The tables of scaled_log_unit (mrg_logtab.h) and sincospi_unit
// (mrg_sincostab.h) in LDS: every kernel whose code evaluates a transform
// stages what it reads once per block with stage_tables() (all threads, then
// a barrier) before any call.
//
// Entries are pairs of doubles, 16 bytes apart, read with one 16-byte load.
// Lanes read them at random; with 16 waves on a CU such a load took 6.5
// cycles a wave, the 24-byte log entries before it (an 8-byte pair load and a
// single) 13, and two doubles 16 bytes apart in a 32-byte entry (the fp32
// sine and cosine) 19: LDS was busy for four fifths of an fp32 normal launch.
// With the shorter functions below (75 -> 72 VALU instructions a pair, 32 -> 30
// an exponential), 2^30 fp64 normals 1771 -> 1620 us, 2^24 fp32 exponentials
// and their substream step 28.0 -> 26.5 us, the paper's 10^8 MRG31k3p normals
// 205 -> 192 us.  Three quarters of an fp64 normal launch is VALU issue.
typedef double double2v __attribute__((ext_vector_type(2)));
constexpr LogTable halved(LogTable t) {
    for (auto& e : t.e) {
        e[0] *= 0.5;
        e[1] *= 0.5;
    }
    return t;
}
static __constant__ LogTable g_logtab = kLogTable;
static __constant__ LogTable g_logtab_half = halved(kLogTable);
static __constant__ SinCosTable g_sincostab = kSinCosTable;

// The log table of SCALE (1 or 2): -SCALE R and SCALE log(R) of every entry.
template <int SCALE>
__device__ __forceinline__ double2v* log_table_lds() {
    __shared__ double2v tab[kLogTabN];
    return tab;
}

__device__ __forceinline__ double2v* sincos_table_lds() {
    __shared__ double2v tab[kSinCosTabN * 2];  // (sin, cos) of each entry, then their low parts
    return tab;
}

// COUNT pairs from constant memory to LDS (and their halves to `half`), one per
// lane, the block's waves in turn.  The loop counter is wave-uniform (readfirstlane): a loop bounded by
// threadIdx and blockDim themselves makes the compiler treat later row
// addresses as divergent.
template <int COUNT>
__device__ __forceinline__ void stage_pairs(double2v* dst, const double (*src)[2], double2v* half = nullptr) {
    const int lane = static_cast<int>(threadIdx.x & 63);
    const int first = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int waves = static_cast<int>(blockDim.x >> 6);
    for (int k = first; k < (COUNT + 63) / 64; k += waves) {
        const int i = lane + 64 * k;
        if (i < COUNT) {
            const double2v v = {src[i][0], src[i][1]};
            dst[i] = v;
            if (half) half[i] = v * 0.5;
        }
    }
}

enum { kStageExponential = 0, kStageNormalF32 = 1, kStageNormal = 2, kStageAll = 3 };
template <int WHAT>
__device__ __forceinline__ void stage_tables() {
    if constexpr (WHAT == kStageExponential) stage_pairs<kLogTabN>(log_table_lds<1>(), g_logtab_half.e);
    if constexpr (WHAT == kStageNormalF32 || WHAT == kStageNormal) stage_pairs<kLogTabN>(log_table_lds<2>(), g_logtab.e);
    // one read for both: a second costs every block its latency again
    if constexpr (WHAT == kStageAll) stage_pairs<kLogTabN>(log_table_lds<2>(), g_logtab.e, log_table_lds<1>());
    if constexpr (WHAT >= kStageNormalF32) stage_pairs<kSinCosTabN>(sincos_table_lds(), g_sincostab.hi);
    if constexpr (WHAT >= kStageNormal) stage_pairs<kSinCosTabN>(sincos_table_lds() + kSinCosTabN, g_sincostab.lo);
    __syncthreads();
}

// x rounded to an integer, as a double and as the low word of the sum that
// rounds it (0 <= x < 2^31): two instructions for both.
__device__ __forceinline__ double round_index(double x_scaled_by, double x, uint32_t* i) {
    const double s = __builtin_fma(x, x_scaled_by, 0x1.8p52);
    *i = static_cast<uint32_t>(__double2loint(s));
    return s - 0x1.8p52;
}

// sin(pi t) and cos(pi t) for t = 2u in (0, 2) (the Box-Muller angle), by
// table: j = rint(128 t) and d = t - j/128 (exact: t and j/128 are within a
// factor of two, or j = 0; |d| <= 1/256); with s_j = sin(pi j/128) and
// c_j = cos(pi j/128) from the table as hi + lo,
// sin(pi t) = s_j + (s_j (cos(pi d) - 1) + c_j sin(pi d))
// and cos(pi t) = c_j + (c_j (cos(pi d) - 1) - s_j sin(pi d)), where
// sin(pi d) runs through d^5 with the d^7 term folded into the lower ones by
// Chebyshev's polynomial on d^2 <= 2^-16 (2^-55 of it is left) and cos(pi d) - 1
// through d^6 (the next term is below 2^-65).  On the axes (j a multiple of
// 64) the table holds exact zeros and ones, so results near the zeros of sin
// and cos keep their relative accuracy.  mrg_transform_accuracy compares both
// results with the HIP library's sincospi over any range of generator
// outputs.
__device__ __forceinline__ void sincospi_unit(double t, double* sp, double* cp) {
    uint32_t j;
    const double jd = round_index(128.0, t, &j);
    const double d = __builtin_fma(jd, -1.0 / 128.0, t);
    const double2v h = sincos_table_lds()[j], l = sincos_table_lds()[kSinCosTabN + j];
    const double z = d * d;
    double ps = 2.550150323800777;                  // pi^5/5! - 3/2 2^-16 pi^7/7!
    ps = __builtin_fma(ps, z, -5.167712779971486);  // -pi^3/3! + 9/16 2^-32 pi^7/7!
    ps = __builtin_fma(ps, z, 3.141592653589793);   // pi
    const double sd = d * ps;
    double pc = -1.3352627688545895;                // -pi^6/6!
    pc = __builtin_fma(pc, z, 4.0587121264167685);  // pi^4/4!
    pc = __builtin_fma(pc, z, -4.934802200544679);  // -pi^2/2!
    const double cm1 = z * pc;
    *sp = h.x + __builtin_fma(h.x, cm1, __builtin_fma(h.y, sd, l.x));
    *cp = h.y + __builtin_fma(h.y, cm1, __builtin_fma(-h.x, sd, l.y));
}

constexpr double kLn2Hi = 6.93147180369123816490e-01;  // ln 2 to 32 bits: k * hi exact
constexpr double kLn2Lo = 1.90821492927058770002e-10;  // ln 2 - hi

// -SCALE log(u), SCALE 1 (exponentials) or 2 (the radius), for the generators'
// uniforms, u in [2^-33, 1) -- never zero, subnormal, negative or non-finite --
// by table: u = m 2^k with m in [1/2, 1); the top 9 fraction bits of m pick an
// interval of width 1/1024 whose entry holds, for SCALE 2, -2 R, R near 1/m
// (R = 1 on the last interval), and 2 log(R) (within 2^-62, and 2^-54 of the
// result).  s = 2 - 2 m R = -2 t with |t| <= 2^-10 (1 + 2^-4), and
// -2 log(m) = 2 log(R) - 2 log1p(t), where log1p(t) = t + t^2 P(t) through t^5
// with the t^6 term folded into P by Chebyshev's polynomial (2^-55 of t is left
// at |t| = 2^-10) and -2 log1p(t) = s + s^2 Q(s).  -2 k ln2_hi + 2 log(R) is
// exact (multiples of 2^-31 and 2^-47 below 2^6).  Near u = 1 (k = 0, R = 1) the
// result is s + s^2 Q(s) alone, accurate relative to its own size.  15
// instructions and one LDS load.
//
// SCALE 1 has half of everything: table, constants and coefficients differ by
// powers of two, so its result is exactly half of SCALE 2's.  With the factor in
// the rate instead, rates above 2^1022, whose reciprocal is subnormal, would lose
// the bit that half of it has no room for.
template <int SCALE>
__device__ __forceinline__ double scaled_log_unit(double u) {
    static_assert(SCALE == 1 || SCALE == 2, "tables of two scales");
    constexpr double f = 2.0 / SCALE;  // s is 1/f of SCALE 2's
    const int k = __builtin_amdgcn_frexp_exp(u);
    const double m = __builtin_amdgcn_frexp_mant(u);  // [1/2, 1)
    static_assert(kLogTabN == 512, "the index takes the top 9 fraction bits of m");
    const uint32_t j = (static_cast<uint32_t>(__double2hiint(m)) >> 11) & (kLogTabN - 1);
    const double2v e = log_table_lds<SCALE>()[j];
    const double s = __builtin_fma(m, e.x, static_cast<double>(SCALE));
    double q = 0x1.999999999999ap-7 * f * f * f * f;               // 1/80
    q = __builtin_fma(q, s, 0x1.00000aaaaaaabp-5 * f * f * f);     // 1/32 + 2^-20/48
    q = __builtin_fma(q, s, 0x1.5555555555555p-4 * f * f);         // 1/12
    q = __builtin_fma(q, s, 0x1.ffffffffffeabp-3 * f);             // 1/4 - 2^-40/96
    const double kd = static_cast<double>(k);
    const double lo = __builtin_fma(s * s, q, kd * (-SCALE * kLn2Lo));
    return __builtin_fma(kd, -SCALE * kLn2Hi, e.y) + (s + lo);
}

// ----------------------------------------------- transforms for fp32 output
// A normal or exponential draw stored as a float needs its value to about
// 1e-7 relative, not to the last bit of a double, so these evaluate the same
// formulas with shorter series and no refinement of the hardware estimates.
// Their results are rounded to float.  Each function's relative error
// (bounds below, checked over every generator output by
// mrg_transform_accuracy) stays under 2e-7.  The largest error of a stored
// float is then under 4e-7 of max(|value|, 1), against the 1e-6 fp32
// tolerance.

// -SCALE log(u) by scaled_log_unit's table: log1p(t) through t^3 (the next term,
// t^4/4 < 2^-41, is below 2^-31 of any result outside the last interval, where
// |log u| >= 2^-10, and of t on the last one); the low bits of ln 2 are left
// out (below 2^-31 of the result).  Near u = 1 (k = 0, R = 1) the result is
// -SCALE log1p(t) alone, accurate relative to its own size.
template <int SCALE>
__device__ __forceinline__ double scaled_log_unit_f32out(double u) {
    constexpr double f = 2.0 / SCALE;
    const int k = __builtin_amdgcn_frexp_exp(u);
    const double m = __builtin_amdgcn_frexp_mant(u);  // [1/2, 1)
    const uint32_t j = (static_cast<uint32_t>(__double2hiint(m)) >> 11) & (kLogTabN - 1);
    const double2v e = log_table_lds<SCALE>()[j];
    const double s = __builtin_fma(m, e.x, static_cast<double>(SCALE));
    const double q = __builtin_fma(s * s, __builtin_fma(s, f * f / 12.0, f / 4.0), s);
    constexpr double kLn2 = 6.93147180559945286227e-01;
    return __builtin_fma(static_cast<double>(k), -SCALE * kLn2, e.y) + q;
}

// sqrt(x) for the radius argument, x in [2^-32, 47]: the hardware reciprocal
// square root and one Newton correction of g = x y (relative error of the
// order of the estimate's square, far below 1e-7).
__device__ __forceinline__ double sqrt_radius_f32out(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double g = x * y;
    const double d = __builtin_fma(-g, g, x);
    return __builtin_fma(d, 0.5 * y, g);
}

// sin(pi t), cos(pi t) by sincospi_unit's table (the high parts only):
// d = t - j/128, |d| <= 1/256, sin(pi d) through d^3 (next term below 2e-10 of
// it) and cos(pi d) - 1 through d^2 (next term below 1e-9 in absolute value;
// beside the zero of cos(pi t) it is scaled by |c_j| <= 0.025, under 4e-9 of
// the result there).  On the axes the table holds exact zeros and ones, so
// results near the zeros of sin and cos keep their relative accuracy.
__device__ __forceinline__ void sincospi_unit_f32out(double t, double* sp, double* cp) {
    uint32_t j;
    const double jd = round_index(128.0, t, &j);
    const double d = __builtin_fma(jd, -1.0 / 128.0, t);
    const double2v h = sincos_table_lds()[j];
    const double z = d * d;
    const double sd = d * __builtin_fma(z, -5.16771278004997, 3.141592653589793);  // pi d - (pi d)^3/6
    const double cm1 = z * -4.934802200544679;                                     // -(pi d)^2/2
    *sp = __builtin_fma(h.y, sd, __builtin_fma(h.x, cm1, h.x));
    *cp = __builtin_fma(-h.x, sd, __builtin_fma(h.y, cm1, h.y));
}

__device__ __forceinline__ double to_f64(uint32_t z) { return static_cast<double>(z); }
__device__ __forceinline__ double to_f64(double z) { return z; }
__device__ __forceinline__ uint32_t to_u32(uint32_t z) { return z; }
__device__ __forceinline__ uint32_t to_u32(double z) { return static_cast<uint32_t>(z); }

}  // namespace mrg355
