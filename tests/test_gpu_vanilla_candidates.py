"""Vanilla candidates come from the embedding lists or from the passages' codes, whichever reads less: both against the oracle,
with passage counts around the 64 that a workgroup of the code form takes and query counts around the 32 of a mask word."""
import pytest

from synth import make_workload, tiny_config

import test_gpu_vanilla as tv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,P,lo,hi,nq", [
    (8, 63, 0, 70, 1),         # long lists: codes; empty passages, passages longer than 64 tokens
    (8, 65, 1, 70, 33),
    (8, 128, 1, 9, 32),
    (3000, 3000, 20, 40, 1),   # short lists of one query: the lists
])
def test_candidates(C, P, lo, hi, nq):
    import paper_2205_09707_amd as pl
    pl.load_library()
    w = make_workload(tiny_config(C=C, P=P, lo=lo, hi=hi, nq=nq, seed=91), noise="calibrated")
    tv._check(pl, w, [(1, 1 << 16, 5), (2, 20, 5)], queries=sorted({0, nq // 2, nq - 1}))
