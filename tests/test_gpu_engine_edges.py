"""GPU parity of one generator step at the edges of its fp64 arithmetic.

The fp64 engine carries each component less h = (m2 - 1)/2, rounds a quotient
to the nearest integer and folds the difference of the components with one
clamp.  Its edges are the residues next to -h, 0 and h (component values 0,
h and m - 1, where the nearest quotient changes), differences next to 0 (where
z wraps to m1) and the largest products (words 0 and m - 1 side by side).
Whole numbers: draws and states must equal the oracle's.
"""
import itertools

import numpy as np
import pytest

import crafted as C
import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2201_06604_amd as P  # noqa: E402


def edge_states(gen):
    """States whose next step makes chosen component values, and states of
    extreme words."""
    (m1, m2), (a1, a2), _ = C.PARAMS[gen]
    h = (m2 - 1) // 2
    rng = np.random.default_rng(17)
    states = []
    for x2 in (0, 1, 2, h - 1, h, h + 1, h + 2, m2 - 2, m2 - 1):
        edges = {0, 1, h - 1, h, h + 1, m1 // 2, m1 // 2 + 1, m1 - 2, m1 - 1, x2, x2 + 1, abs(x2 - 1)}
        for x1 in edges:  # undo one step that made (x1, x2)
            c1 = tuple(int(v) for v in rng.integers(0, m1, size=2)) + (x1,)
            c2 = tuple(int(v) for v in rng.integers(0, m2, size=2)) + (x2,)
            states.append(C._to_external(gen, C._undo(c1, a1, m1), C._undo(c2, a2, m2)))
    words1, words2 = (0, h, m1 - 1), (0, h, h + 1, m2 - 1)
    for c1 in itertools.product(words1, repeat=3):
        for c2 in itertools.product(words2, repeat=3):
            if any(c1) and any(c2):
                states.append(list(c1) + list(c2))
    return C.records(np.array(states, dtype=np.uint32))


@pytest.mark.parametrize("gen", [P.MRG_GEN_MRG32K3A, P.MRG_GEN_MRG31K3P])
@pytest.mark.parametrize("draws,chunk", [(1, 0), (5, 0), (7, 3)])
def test_step_at_the_edges(gen, draws, chunk):
    rec = edge_states(gen)
    n = rec.shape[0] * draws
    d = torch.from_numpy(rec.view(np.int32).copy()).cuda()
    got = P.as_u32(P.mrg_generate(d, n, P.MRG_RAW, P.MRG_U32, gen=gen, cfg=dict(chunk=chunk) if chunk else None))
    want_rec = rec.copy()
    want = O.generate(gen, want_rec, n, O.RAW, O.U32)
    np.testing.assert_array_equal(got[:n], want)
    np.testing.assert_array_equal(P.as_u32(d), want_rec)
