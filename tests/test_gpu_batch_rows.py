"""Batch plans whose gangs hold whole rows: a request's stream blocks share one
gang, two a wave where they outnumber its waves, cut into column groups above
that.  Stream counts at the edges of waves, gangs and column groups, ragged draw
counts, one and several chunks per stream; every request equals its own plain
launch bit for bit, outputs and states, and nothing past an output is written.
"""
import numpy as np
import pytest

import oracle as O
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2201_06604_amd as P  # noqa: E402

KINDS = [(P.MRG_UNIFORM, P.MRG_F64), (P.MRG_UNIFORM, P.MRG_F32), (P.MRG_RAW, P.MRG_U32), (P.MRG_NORMAL, P.MRG_F64),
         (P.MRG_NORMAL, P.MRG_F32), (P.MRG_EXPONENTIAL, P.MRG_F64), (P.MRG_EXPONENTIAL, P.MRG_F32)]
TORCH = {P.MRG_F64: torch.float64, P.MRG_F32: torch.float32, P.MRG_U32: torch.int32}


def requests(counts, draws):
    """(streams, n, dist, dtype), the kinds in turn; n leaves some streams a draw more."""
    return [(S, S * draws + (7 * i) % S, *KINDS[i % len(KINDS)]) for i, S in enumerate(counts)]


def check(reqs, cfg):
    total = sum(r[0] for r in reqs)
    rec = O.create_streams(1, workloads.random_seed(31), total).view(np.int32)
    mine, plain = torch.from_numpy(rec.copy()).cuda(), torch.from_numpy(rec.copy()).cuda()
    outs, args, first = [], [], 0
    for S, n, dist, dtype in reqs:
        out = torch.full((n + 64,), 7, dtype=TORCH[dtype], device="cuda")
        args.append(P.make_request(mine[first:first + S], n, dist, dtype, 0.75, out))
        outs.append(out)
        first += S
    plan = P.BatchPlan(args, cfg=cfg)
    plan.upload()
    plan.launch()
    first = 0
    for out, (S, n, dist, dtype) in zip(outs, reqs):
        want = P.mrg_generate(plain[first:first + S], n, dist, dtype, 0.75)
        assert torch.equal(out[:n], want[:n]), (S, n, dist, dtype, cfg)
        assert bool((out[n:] == 7).all()), (S, n, dist, dtype, cfg)
        first += S
    assert torch.equal(mine, plain), cfg


EDGES = [1, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 575, 576, 577, 640, 641, 1000, 1023, 1024, 1025,
         1087, 1600, 2047, 2048, 2049]


@pytest.mark.parametrize("draws,tile", [(1, 0), (7, 0), (100, 0), (101, 32), (64, 3)])
@pytest.mark.parametrize("gang", [0, 2, 4])
def test_rows_at_the_edges(gang, draws, tile):
    for shift in range(0, len(KINDS), 3):  # other kinds for each stream count
        check(requests(EDGES[shift:] + EDGES[:shift], draws), dict(gang_waves=gang, tile_units=tile))


@pytest.mark.parametrize("n_req", [1, 3, 40, 300])
def test_automatic_tile_lengths(n_req):
    """Mixes of little and of much work, whose automatic tiles have other lengths."""
    rng = np.random.default_rng(n_req)
    counts = rng.integers(1, 1400, n_req)
    reqs = [(int(S), int(10 ** rng.uniform(0, 6)), *KINDS[int(rng.integers(len(KINDS)))]) for S in counts]
    check(reqs, None)
