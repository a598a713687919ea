"""mrg_batch_autotune times the plan's own shape beside its candidates, so that a plan is
not exchanged for a slower one: with room for no other shape it times and keeps its own.
"""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2201_06604_amd as P  # noqa: E402


def make(n_req, S, n, cfg):
    streams = P.mrg_streams_create_device(P.mrg_creator_init([12345] * 6), n_req * S)
    outs = [torch.zeros(n, dtype=torch.float32, device="cuda") for _ in range(n_req)]
    reqs = [P.make_request(streams[S * i:S * i + S], n, P.MRG_UNIFORM, P.MRG_F32, 1.0, outs[i]) for i in range(n_req)]
    return P.BatchPlan(reqs, cfg=cfg), streams, outs


def tune(plan, room):
    ws = torch.zeros(room, dtype=torch.uint8, device="cuda")
    best, ms = P.mrg_batch_cfg(), ctypes.c_double()
    P._check(P.lib().mrg_batch_autotune(plan._p, ctypes.c_void_p(ws.data_ptr()), room, None, ctypes.byref(best),
                                        ctypes.byref(ms)))
    return best, ms.value


def test_own_shape_is_timed_where_no_other_fits():
    plan, streams, _ = make(40, 64, 64 * 100_000, dict(tile_units=100_000, gang_waves=8))  # one tile a request
    before = streams.clone()
    best, ms = tune(plan, plan.workspace_size())
    assert ms > 0.0 and (best.tile_units, best.gang_waves) == (100_000, 8)
    assert torch.equal(streams, before)
