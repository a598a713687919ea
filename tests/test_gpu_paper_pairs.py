"""The two-dimensional placement with pairs stored together (even row stride,
output aligned to a pair) and one by one: the same numbers and states bit for bit,
and nothing written beside the block.  Visit counts of every remainder of three, few
and many rows, one row cut into column blocks; every distribution and type.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2201_06604_amd as P  # noqa: E402

KINDS = [(P.MRG_UNIFORM, P.MRG_F64), (P.MRG_UNIFORM, P.MRG_F32), (P.MRG_RAW, P.MRG_U32), (P.MRG_NORMAL, P.MRG_F64),
         (P.MRG_NORMAL, P.MRG_F32), (P.MRG_EXPONENTIAL, P.MRG_F64), (P.MRG_EXPONENTIAL, P.MRG_F32)]
TORCH = {P.MRG_F64: torch.float64, P.MRG_F32: torch.float32, P.MRG_U32: torch.int32}


def block(rec, nrow, ncol, npad, first, G0, G1, dist, dtype, gen):
    """The block, from an output that starts `first` elements into its buffer."""
    flat = torch.full((first + nrow * npad + 64,), 7, dtype=TORCH[dtype], device="cuda")
    s = rec.clone()
    out = flat[first:first + nrow * npad].view(nrow, npad)
    P.mrg_generate_paper(s, nrow, ncol, G0, G1, dist, dtype, 0.75, out=out, npad=npad, gen=gen)
    assert bool((flat[:first] == 7).all()) and bool((flat[first + nrow * npad:] == 7).all())
    assert bool((out[:, ncol:] == 7).all())
    return out[:, :ncol].clone(), s


@pytest.mark.parametrize("gen", [P.MRG_GEN_MRG32K3A, P.MRG_GEN_MRG31K3P])
@pytest.mark.parametrize("nrow,G0", [(1, 1), (3, 2), (257, 64), (40, 8)])
def test_pairs_together_and_apart_agree(gen, nrow, G0):
    for G1, ncol in [(2, 2), (2, 14), (16, 46), (16, 80), (64, 62), (64, 4100), (6, 6 * 31 + 2)]:
        rec = P.mrg_streams_create_device(P.mrg_creator_init([77] * 6, gen=gen), G0 * G1, gen=gen)
        for dist, dtype in KINDS:
            want, states = block(rec, nrow, ncol, ncol + 1, 0, G0, G1, dist, dtype, gen)  # odd stride: one by one
            for npad, first in [(ncol, 0), (ncol + 2, 0), (ncol, 1), (ncol, 2)]:
                got, after = block(rec, nrow, ncol, npad, first, G0, G1, dist, dtype, gen)
                assert torch.equal(got, want), (G1, ncol, dist, dtype, npad, first)
                assert torch.equal(after, states), (G1, ncol, dist, dtype, npad, first)
