"""Vanilla candidates come from the embedding lists or from the passages' codes, whichever reads less: both against the oracle,
with passage counts around the 64 that a workgroup of the code form takes and query counts around the 32 of a mask word.
Which of the two a case takes is worked out here by the rule of k_vanilla.hip and part of the test."""
import numpy as np
import pytest

from oracle import oracle as orc
from synth import make_workload, tiny_config

import parity_util as pu
import test_gpu_vanilla as tv

pytestmark = pytest.mark.gpu
UNIT, THREADS, WAVE = 512, 256, 64  # van_probe_mask_kernel: entries per unit of work, threads per query, per wave


def _by_codes(w, nprobe):
    """True: from the codes.  None: the masks have no room, the lists are walked without a decision."""
    ix = pu.oracle_index(w)
    nq, N = w.queries.shape[0], w.N
    masks = (nq + 31) // 32
    if ix.C * masks > 2 * nq * w.cfg.P:
        return None
    length = np.bincount(ix.codes, minlength=ix.C)
    units = 0
    for q in range(nq):
        probed = np.unique(orc.top_nprobe(orc.scq(ix.centroids, w.queries[q].numpy()), nprobe))
        entries = np.zeros(THREADS // WAVE, np.int64)
        for u, c in enumerate(probed):
            entries[u % THREADS // WAVE] += length[c]
        units += int(((entries + UNIT - 1) // UNIT).sum())
    return units * UNIT > N // 4 * masks


@pytest.mark.parametrize("C,P,lo,hi,nq,zipf,by_codes", [
    (8, 63, 0, 70, 1, 1.1, True),         # long lists; empty passages, passages longer than 64 tokens
    (8, 65, 1, 70, 33, 1.1, True),
    (8, 128, 1, 9, 32, 1.1, True),
    (3000, 3000, 20, 40, 1, 1.1, True),   # the centroids of most tokens are popular ones
    (3000, 3000, 20, 40, 1, 0.0, False),  # as many passages per centroid everywhere: short lists
    (8192, 3000, 20, 40, 33, 0.0, False),
    (200, 90, 1, 9, 1, 1.1, None),
])
def test_candidates(C, P, lo, hi, nq, zipf, by_codes):
    import paper_2205_09707_amd as pl
    pl.load_library()
    w = make_workload(tiny_config(C=C, P=P, lo=lo, hi=hi, nq=nq, seed=91, zipf_s=zipf), noise="calibrated")
    for nprobe in (1, 2):
        assert _by_codes(w, nprobe) is by_codes, nprobe
    tv._check(pl, w, [(1, 1 << 16, 5), (2, 20, 5)], queries=sorted({0, nq // 2, nq - 1}))


def test_both_sides_of_the_rule():
    """One query with one more probe at a time, until its lists hold more than a quarter of the tokens."""
    import paper_2205_09707_amd as pl
    pl.load_library()
    w = make_workload(tiny_config(C=512, P=3000, lo=20, hi=40, nq=1, seed=92, zipf_s=0.0), noise="calibrated")
    sides = [_by_codes(w, nprobe) for nprobe in range(1, 9)]
    assert sides == sorted(sides) and sides[0] is False and sides[-1] is True, sides
    first = sides.index(True) + 1  # the smallest nprobe that takes the codes
    tv._check(pl, w, [(nprobe, 1 << 16, 5) for nprobe in (first - 1, first)] + [(nprobe, 100, 5) for nprobe in (first - 1, first)])
