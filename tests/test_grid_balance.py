"""Automatic launches come out evenly over the 256 CUs for any stream count, not for
powers of two alone: the plan's blocks, dealt in turn to the CU with the least work,
leave the busiest CU within about a third of the mean (a last round of few blocks after
three full ones; a round of few blocks after one would be twice the mean).  Host only.
From 2^27 draws on, where the launch lasts long enough that nothing else decides, and
from two waves a SIMD on.
"""
import heapq

import pytest

import paper_2201_06604_amd as P
from paper_2201_06604_amd import tune_plain as T


def busiest_over_mean(plan, S, units):
    """(waves of the grid, work of the busiest CU over the mean of the CUs)."""
    n_sblk = -(-S // (64 * plan["streams_per_lane"]))
    wpb, chunks = plan["block"] // 64, -(-units // plan["chunk"])
    if not plan["lockstep"] and 1 < chunks <= wpb:  # a column: a stream block's chunks in one block
        blocks = [units] * n_sblk
    else:
        blocks = []
        for j in range(chunks):
            u = min(plan["chunk"], units - j * plan["chunk"])
            full, rest = divmod(n_sblk, wpb)
            blocks += [wpb * u] * full + [rest * u] * (rest > 0)
    cus = [0] * 256
    for b in blocks:
        heapq.heapreplace(cus, cus[0] + b)
    return n_sblk * chunks, max(cus) / (sum(cus) / 256)


@pytest.mark.parametrize("kind", range(len(T.KINDS)), ids=[k[0] for k in T.KINDS])
@pytest.mark.parametrize("n", [1 << 27, 1 << 28, 1 << 30])
def test_busiest_cu_is_close_to_the_mean(kind, n):
    _, dist, dtype = T.KINDS[kind]
    uneven = []
    for S in range(2048, 262145, 64 * 7):  # every residue of the blocks' widths
        per = n // S
        plan = P.mrg_generate_plan(S, per * S, dist, dtype)
        waves, load = busiest_over_mean(plan, S, -(-per // 2) if dist == P.MRG_NORMAL else per)
        if waves >= 2048 and load > 1.35:
            uneven.append((S, round(load, 3), plan))
    assert not uneven, uneven[:5]


def test_mostly_idle_last_blocks_get_many_chunks():
    """Rows in step on shared lines, of 9 and of 36 stream blocks: one round of blocks of
    16 waves would hold 9 live ones, or leave a third of the CUs with four."""
    for S in (555, 2252):
        plan = P.mrg_generate_plan(S, 1 << 28, P.MRG_UNIFORM, P.MRG_F32)
        chunks = -(-((1 << 28) // S + 1) // plan["chunk"])
        assert plan["lockstep"] and -(-S // 64) * chunks >= 16384, plan


@pytest.mark.parametrize("dtype", [P.MRG_F64, P.MRG_F32])
@pytest.mark.parametrize("S", [64, 77, 128])
def test_short_normals_stage_their_tables_by_four_waves(S, dtype):
    """Rows that fit in one block may take a block of one or two waves; calls of normals
    too short to spread the staging of the tables keep four."""
    for n in (1 << 22, 1 << 23, 1 << 24, (1 << 26) - 64):
        plan = P.mrg_generate_plan(S, n // S * S, P.MRG_NORMAL, dtype)
        assert plan["block"] >= 256, (n, plan)
