"""Automatic launches whose chunks and block widths are chosen by the grid they make,
and the XCD order of any number of blocks, against the one-chunk launch of the same
call: outputs and states bit for bit, nothing past the output written.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2201_06604_amd as P  # noqa: E402
from test_gpu_columns import KINDS, check  # noqa: E402

GEN = P.MRG_GEN_MRG32K3A


# rows on pages, on lines and anywhere; a few stream blocks, many, and one more than a round of blocks
@pytest.mark.parametrize("S", [64, 77, 555, 640, 2252, 9984, 10240, 20032, 131072, 131136])
@pytest.mark.parametrize("n", [(1 << 22) + 12345, (1 << 26) + 54321])
def test_chosen_grids_and_one_chunk_agree(S, n):
    check(GEN, S, n // S * S if S % 64 == 0 else n, KINDS, None, calls=1)


@pytest.mark.parametrize("lockstep", [0, 1])
@pytest.mark.parametrize("blocks", [1, 7, 9, 63, 65])
def test_xcd_order_of_any_number_of_blocks(blocks, lockstep):
    S = 64 * 4 * blocks - 3  # blocks of 4 waves, one chunk; then three chunks each
    check(GEN, S, S * 30 + 5, KINDS[::2], dict(block=256, chunk=1 << 20, xcd_remap=1, lockstep=lockstep), calls=1)
    check(GEN, S, S * 60 + 5, KINDS[::2], dict(block=256, chunk=5, xcd_remap=1, lockstep=lockstep), calls=1)
