"""Column launches of mrg_generate (all of a stream block's chunks in one block,
which writes the states back itself) and the automatic shapes around them, against
the one-chunk launch of the same call: outputs and states bit for bit, nothing past
the output written.  Stream counts at the edges of a wave, ragged and odd draw
counts, calls shorter than the streams, two to sixteen chunks and one more than a
column holds; repeated calls, so that a wrong state shows in the next one.
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


def check(gen, S, n, kinds, cfg, calls=2):
    rec = O.create_streams(gen, workloads.random_seed(11), S).view(np.int32)
    for dist, dtype in kinds:
        mine, plain = torch.from_numpy(rec.copy()).cuda(), torch.from_numpy(rec.copy()).cuda()
        for _ in range(calls):
            out = torch.full((n + 64,), 7, dtype=TORCH[dtype], device="cuda")
            want = torch.full((n + 64,), 7, dtype=TORCH[dtype], device="cuda")
            P.mrg_generate(mine, n, dist, dtype, 0.75, out=out, gen=gen, cfg=cfg)
            P.mrg_generate(plain, n, dist, dtype, 0.75, out=want, gen=gen, cfg=dict(block=64, chunk=1 << 30))
            assert torch.equal(out, want), (gen, S, n, dist, dtype, cfg)
            assert torch.equal(mine, plain), (gen, S, n, dist, dtype, cfg)


@pytest.mark.parametrize("gen", [P.MRG_GEN_MRG32K3A, P.MRG_GEN_MRG31K3P])
@pytest.mark.parametrize("S", [1, 63, 64, 65, 128, 1000])
def test_columns_and_one_chunk_agree(gen, S):
    for draws in (1, 2, 5, 47, 64, 65):
        for n in {max(1, S * draws - S // 2), S * draws, S * draws + 1, S * draws + S // 3}:
            check(gen, S, n, KINDS, dict(block=1024, chunk=4))  # up to 17 chunks: 16 make a column
            check(gen, S, n, KINDS[::3], dict(block=128, chunk=(draws + 1) // 2))


@pytest.mark.parametrize("spl", [2, 4])
@pytest.mark.parametrize("xcd", [0, 1])
def test_columns_of_several_streams_a_lane(spl, xcd):
    for S in (64 * spl, 64 * spl * 8, 64 * spl * 8 + spl, 500):
        for n in (S * 30, S * 30 + 5, S * 7 - 1):
            check(P.MRG_GEN_MRG32K3A, S, n, KINDS, dict(block=512, chunk=4, streams_per_lane=spl, xcd_remap=xcd))


# on both sides of each class and half, few and many streams, rows on lines and not
@pytest.mark.parametrize("n", [1 << 10, 1 << 15, (1 << 15) - 7, 1 << 18, 1 << 20, 1 << 22, 23_726_566, 1 << 26])
def test_automatic_shapes_and_one_chunk_agree(n):
    for S in (64, 1001, 16384, 100003):
        check(P.MRG_GEN_MRG32K3A, S, n, KINDS, None, calls=1)


# rows in step that share lines: 16, 1,023 and 1,024 stream blocks, where the aim changes
@pytest.mark.parametrize("S", [1001, 65471, 65473])
def test_rows_in_step_and_one_chunk_agree(S):
    check(P.MRG_GEN_MRG32K3A, S, (1 << 26) + 12345, KINDS, None, calls=1)
