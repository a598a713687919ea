"""The workspace of automatic batch plans near the size of the static one: shorter
automatic tiles and the requests' own records must not push out a plan that tiles of
256 units leave room for.  Host only; pointers are never followed.
"""
import ctypes

import paper_2201_06604_amd as P


def workspace(reqs, cfg=None):
    arr = (P.mrg_request * len(reqs))(*reqs)
    plan, size = ctypes.c_void_p(), ctypes.c_size_t()
    c = None if cfg is None else ctypes.byref(P.mrg_batch_cfg(*cfg))
    assert P.lib().mrg_batch_plan_create(1, arr, len(reqs), c, ctypes.byref(plan)) == 0
    assert P.lib().mrg_batch_workspace_size(plan, ctypes.byref(size)) == 0
    P.lib().mrg_batch_plan_destroy(plan)
    return size.value


def mix(small, big):
    """`small` requests of one draw a stream and `big` of 4,096 draws from 1,024 streams."""
    reqs, streams, out = [], 1 << 20, 1 << 34
    for S, per, k in ((64, 1, small), (1024, 4096, big)):
        for _ in range(k):
            reqs.append(P.mrg_request(streams, S, S * per, P.MRG_UNIFORM, P.MRG_F32, 1.0, out))
            streams += S * 72
            out += S * per * 4
    return reqs


def test_plans_that_fit_the_static_workspace_still_do():
    # 136 bytes a small request (its slot, record and tile) and 80 large ones: 15.95 MiB
    reqs = mix(120_500, 80)
    assert workspace(reqs) <= P.MRG_BATCH_STATIC_WORKSPACE_BYTES
    # a little batch keeps its short tiles and the larger workspace that they take
    assert workspace(mix(10, 80)) > workspace(mix(10, 80), (256, 0, 0, 0))
