"""Write mrg_logtab.h: the 512-entry table of scaled_log_unit (mrg_engine.h).

    python paper_2201_06604_amd/csrc/gen_logtab.py

A uniform u = m 2^k (m in [1/2, 1)) falls in interval j = floor(1024 (m - 1/2))
of width 1/1024 (the top 9 fraction bits of m).  With R_j near 1/c_j (c_j the
interval's midpoint) and t = m R_j - 1, |t| <= 2^-10 (1 + 2^-4),
  -2 log(u) = -2 k ln2 + 2 log(R_j) - 2 log1p(t).
Entry j holds -2 R_j (so that one FMA gives -2 t) and the multiple of 2^-47
nearest 2 log(R_j), which -2 k ln2_hi can be added to exactly.  No low part is
stored: among the multiples of 2^-32 within 2^17 2^-32 of 1/c_j, R_j is the
one whose logarithm lies nearest a multiple of 2^-48 -- within 2^-54 of the
smallest |log(u)| of its interval and within 2^-63 (both checked below).  The
last interval has R = 1, so that t = m - 1 near u = 1.

The search evaluates log((n + i) 2^-32) = log(n 2^-32) + log1p(i/n) in units of
2^-90, modulo 2^-48; what it finds is checked with Python's decimal module at
60 significant digits.
"""
import os
from decimal import Decimal, getcontext

import numpy as np

getcontext().prec = 60
HERE = os.path.dirname(os.path.abspath(__file__))
N = 512
REACH = 1 << 17


def nearest_r(c: Decimal) -> Decimal:
    """The R of an interval with midpoint c."""
    n = int((Decimal(2) ** 32 / c).to_integral_value())
    i = np.arange(-REACH, REACH + 1, dtype=np.int64)
    unit = Decimal(2) ** 90
    base = int(((Decimal(n) / Decimal(2) ** 32).ln() * unit).to_integral_value()) % (1 << 64)
    first = int((unit / n).to_integral_value()) % (1 << 64)
    x = i / float(n)
    rest = (x * x * (-1 / 2 + x * (1 / 3 - x / 4)) * 2.0 ** 90).astype(np.int64)
    with np.errstate(over="ignore"):
        at = np.uint64(base) + i.astype(np.uint64) * np.uint64(first) + rest.astype(np.uint64)
    off = (at & np.uint64((1 << 42) - 1)).astype(np.int64)  # modulo 2^-48
    off = np.minimum(off, (1 << 42) - off)
    return Decimal(n + int(i[off.argmin()])) / Decimal(2) ** 32


def entries():
    out = []
    for j in range(N):
        m_lo = Decimal(1) / 2 + Decimal(j) / 1024
        m_hi = m_lo + Decimal(1) / 1024
        r = Decimal(1) if j == N - 1 else nearest_r((m_lo + m_hi) / 2)
        v = r.ln()
        hi = (v * Decimal(2) ** 48).to_integral_value() / Decimal(2) ** 48
        assert abs(v - hi) <= min(Decimal(2) ** -54 * -m_hi.ln(), Decimal(2) ** -63), (j, v - hi)
        assert max(abs(m_lo * r - 1), abs(m_hi * r - 1)) <= Decimal(2) ** -10 * (1 + Decimal(2) ** -4), j
        out.append((float(-2 * r), float(2 * hi)))
        assert Decimal(out[-1][0]) == -2 * r and Decimal(out[-1][1]) == 2 * hi
    return out


def main():
    rows = [f"    {{{r.hex()}, {hi.hex()}}},  // j = {j}" for j, (r, hi) in enumerate(entries())]
    text = """// mrg_logtab.h -- table of scaled_log_unit (mrg_engine.h): for interval j of the
// mantissa m in [1/2, 1) (m in [1/2 + j/1024, 1/2 + (j+1)/1024)), -2 R and
// 2 log(R), R near the reciprocal of the interval's midpoint and chosen so that
// log(R) lies within 2^-63 of the multiple of 2^-48 stored (R = 1 for the last
// one).  Written by gen_logtab.py (checked with Python decimal arithmetic at 60
// digits); do not edit.
#pragma once

namespace mrg355 {

constexpr int kLogTabN = %d;
struct LogTable {
    double e[kLogTabN][2];  // (-2 R, 2 log R) of each interval
};
constexpr LogTable kLogTable = {{
%s
}};

}  // namespace mrg355
""" % (N, "\n".join(rows))
    with open(os.path.join(HERE, "mrg_logtab.h"), "w") as f:
        f.write(text)


if __name__ == "__main__":
    main()
