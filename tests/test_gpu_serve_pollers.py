"""Requests answered while other threads poll a finished one in a loop: the scheduler
gives way to as many calls as are waiting, not until none is, so launches and
completions go on; every output equals its session's draws from the request's offset
on, bit for bit.
"""
import threading
import time

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2201_06604_amd as P  # noqa: E402

SEED = [21, 22, 23, 24, 25, 26]


@pytest.mark.parametrize("pollers,mode", [(1, 0), (4, 0), (4, 1)])
def test_requests_are_answered_beside_threads_that_poll(pollers, mode):
    pool = torch.zeros(64 << 20, dtype=torch.uint8, device="cuda")
    srv = P.Server(8, SEED, pool, mode=mode)
    first, _ = srv.submit(7, 1000, P.MRG_UNIFORM, P.MRG_F64, 1.0)
    while not srv.poll(first)[0]:
        time.sleep(0)
    stop, polls = threading.Event(), [0] * pollers

    def poll(k):
        while not stop.is_set():
            assert srv.poll(first)[0]
            polls[k] += 1

    ts = [threading.Thread(target=poll, args=(k,)) for k in range(pollers)]
    [t.start() for t in ts]
    got = []
    try:
        end = time.monotonic() + 60
        for r in range(60):
            asked = [(srv.submit(s, 5000 + r + s, P.MRG_NORMAL, P.MRG_F64, 1.0), s, 5000 + r + s) for s in range(1 + r % 7)]
            for (ticket, offset), s, n in asked:
                done, ptr, _ = srv.poll(ticket)
                while not done:
                    assert time.monotonic() < end, "a request was not answered"
                    time.sleep(0)
                    done, ptr, _ = srv.poll(ticket)
                if r % 20 == 0:
                    at = ptr - pool.data_ptr()
                    got.append((s, n, offset, pool[at:at + 8 * n].clone()))
                    torch.cuda.synchronize()
                srv.release(ticket)
    finally:
        stop.set()
        [t.join() for t in ts]
    assert all(polls)
    srv.close()
    streams = P.mrg_streams_create_device(P.mrg_creator_init(SEED), 64 * 8)
    for s, n, offset, data in got:
        mine = streams[64 * s:64 * s + 64].clone()
        P.mrg_streams_advance(mine, offset)
        want = P.mrg_generate(mine, n, P.MRG_NORMAL, P.MRG_F64)
        assert torch.equal(data.view(torch.float64), want[:n]), (s, n, offset)
