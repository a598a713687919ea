"""Requests from several threads at once: each thread submits to sessions of its
own, polls and releases while the others do, and every output equals the draws of
its session's streams from the request's offset on, bit for bit.
"""
import threading
import time

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2201_06604_amd as P  # noqa: E402

KINDS = [(P.MRG_UNIFORM, P.MRG_F64), (P.MRG_UNIFORM, P.MRG_F32), (P.MRG_RAW, P.MRG_U32), (P.MRG_NORMAL, P.MRG_F64),
         (P.MRG_NORMAL, P.MRG_F32), (P.MRG_EXPONENTIAL, P.MRG_F64), (P.MRG_EXPONENTIAL, P.MRG_F32)]
TORCH = {P.MRG_F64: torch.float64, P.MRG_F32: torch.float32, P.MRG_U32: torch.int32}
SEED = [11, 12, 13, 14, 15, 16]
SIZES = [1, 63, 64, 65, 1000, 6145, 20011, 100003]


@pytest.mark.parametrize("threads,lanes", [(1, 1), (3, 4), (6, 2)])
def test_threads_get_their_own_draws(threads, lanes):
    per = 4  # sessions of a thread
    pool = torch.zeros(64 << 20, dtype=torch.uint8, device="cuda")
    srv = P.Server(threads * per, SEED, pool, lanes=lanes)
    got, failed = [[] for _ in range(threads)], []

    def work(k):
        try:
            for rep in range(3):
                asked = []
                for j, n in enumerate(SIZES):
                    sess = k * per + j % per
                    dist, dtype = KINDS[(j + rep + k) % len(KINDS)]
                    ticket, offset = srv.submit(sess, n, dist, dtype, 0.75)
                    asked.append((ticket, sess, n, dist, dtype, offset))
                for ticket, sess, n, dist, dtype, offset in asked:
                    done, ptr, _ = srv.poll(ticket)
                    while not done:
                        time.sleep(0)
                        done, ptr, _ = srv.poll(ticket)
                    size = n * (8 if dtype == P.MRG_F64 else 4)
                    at = ptr - pool.data_ptr()
                    got[k].append((sess, n, dist, dtype, offset, pool[at:at + size].clone()))
                    torch.cuda.synchronize()
                    srv.release(ticket)
        except Exception as e:  # noqa: BLE001
            failed.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(threads)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    srv.close()
    assert not failed, failed
    first = P.mrg_streams_create_device(P.mrg_creator_init(SEED), 64 * threads * per)
    for sess, n, dist, dtype, offset, data in (g for k in got for g in k):
        s = first[64 * sess:64 * sess + 64].clone()
        P.mrg_streams_advance(s, offset)
        want = P.mrg_generate(s, n, dist, dtype, 0.75)
        assert torch.equal(data.view(TORCH[dtype]), want[:n]), (sess, n, dist, dtype, offset)
