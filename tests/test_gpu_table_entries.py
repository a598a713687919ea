"""GPU parity of single table entries where the entry search changes its way.

An entry is searched from a start below the mean with bounds on every rounding,
and decided by the definition where the bounds leave it open: uniforms next to 0
(below the start), next to 1, and on a step of the distribution function.  The
uniforms come from crafted states (tests/crafted.py).  Windows of tables whose
totals stay below 1,024 take their logarithms and entries from on-chip memory,
others from global memory; both, and the totals on either side, are here.  Whole
numbers and table look-ups: everything must equal the oracle's.
"""
import numpy as np
import pytest

import crafted as C
import oracle as O
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2201_06604_amd as P  # noqa: E402


def run(gen, rec, I, J, rows, cols):
    """Everything equals the oracle's; a table of bad margins has zeros, a NaN
    statistic and its stream unmoved (the oracle takes only good ones)."""
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    d = dev(rec.view(np.int32).copy())
    tabs, stats = P.mrg_tables_sample(d, dev(I), dev(J), dev(rows), dev(cols), stats=True, gen=gen)
    n = I.shape[0]
    good = (rows.sum(1) == cols.sum(1)) & (rows.min(1) >= 0) & (cols.min(1) >= 0)
    work, part = rec.copy(), rec[good].copy()
    wtabs, wstats = np.zeros((n, 5, 5), np.int32), np.full(n, np.nan)
    if good.any():
        wtabs[good], wstats[good] = O.tables(gen, part, I[good], J[good], rows[good], cols[good])
        work[good] = part
    np.testing.assert_array_equal(tabs[:n].cpu().numpy(), wtabs)
    np.testing.assert_array_equal(stats[:n].cpu().numpy(), wstats)
    np.testing.assert_array_equal(P.as_u32(d), work)


def two_by_two(rows, cols):
    I = np.full(len(rows), 2, np.int32)
    r, c = np.zeros((len(rows), 5), np.int32), np.zeros((len(rows), 5), np.int32)
    r[:, :2], c[:, :2] = rows, cols
    return I, I.copy(), r, c


@pytest.mark.parametrize("gen", [P.MRG_GEN_MRG32K3A, P.MRG_GEN_MRG31K3P])
@pytest.mark.parametrize("margins", [
    (1, 1, 1, 1), (2, 2, 2, 2), (3, 1, 2, 2), (40, 3, 21, 22),  # steps at simple fractions
    (500, 500, 500, 500), (500, 523, 1000, 23), (511, 512, 3, 1020),  # total 1,000 and 1,023
    (512, 512, 500, 524), (9000, 3900, 178, 12722), (1 << 19, 1 << 19, 1 << 19, 1 << 19),  # 1,024 and above
    (1, (1 << 20) - 1, 700000, 348576)], ids=str)
def test_entries_at_the_ends_and_on_steps(gen, margins):
    m1 = C.modulus1(gen)
    zs = [1, 2, 3, 1000, m1 - 1000, m1 - 2, m1 - 1, m1]
    zs += [k * ((m1 + 1) // 16) + d for k in range(1, 16) for d in (-1, 0, 1)]  # u = k/16, exactly
    rng = np.random.default_rng(sum(margins))
    rec = C.records([C.state_with_outputs(gen, [z], rng) for z in zs])
    r0, r1, c0, c1 = margins
    run(gen, rec, *two_by_two([(r0, r1)] * len(zs), [(c0, c1)] * len(zs)))


@pytest.mark.parametrize("n", [1, 63, 64, 65, 257, 700])
@pytest.mark.parametrize("odd", [None, (1023, 0), (1024, 0), (40000, 0), (40000, 1), (-3, 1)], ids=str)
def test_windows_of_small_and_large_totals(n, odd):
    """One table of the window has total odd[0], or margins that disagree by odd[1]."""
    gen = P.MRG_GEN_MRG32K3A
    I, J, rows, cols = workloads.contingency_margins(n, rng_seed=n)
    if odd:
        k = n // 2
        I[k], J[k] = 2, 2
        rows[k], cols[k] = 0, 0
        rows[k, :2] = (odd[0] // 3, odd[0] - odd[0] // 3)
        cols[k, :2] = (odd[0] // 2 + odd[1], odd[0] - odd[0] // 2)
    run(gen, O.create_streams(gen, workloads.random_seed(n), n), I, J, rows, cols)


def test_windows_of_two_groups_a_wave():
    """The smallest count that takes the wide windows, and a ragged last one."""
    gen, n = P.MRG_GEN_MRG32K3A, 512 * 1024 + 77
    I, J, rows, cols = workloads.contingency_margins(n, rng_seed=9, dim_hi=3, tot_hi=40)
    run(gen, O.create_streams(gen, workloads.random_seed(9), n), I, J, rows, cols)
