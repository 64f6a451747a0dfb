"""The inverted stage-2 kernel scores only the passages whose bound reaches the best ndocs scores seen so far: what it keeps
must be the oracle's ndocs best whatever the number of survivors (bit planes of 31, 36 and 63 slots, and beyond), of
passages (128- and 2048-passage steps, ragged ends, several steps per wave) and of queries (their order over the XCDs)."""
import numpy as np
import pytest

from oracle import oracle as orc
from synth import make_workload, tiny_config

import test_gpu_parity as tp

pytestmark = pytest.mark.gpu

CASES = [
    # C, P, lo, hi, queries, seed: one or several ranges, ragged or not
    (400, 127, 1, 9, 1, 41),
    (400, 128, 1, 9, 7, 42),
    (400, 2049, 1, 9, 9, 43),
    (300, 8192, 2, 12, 8, 44),
    (300, 140_001, 2, 6, 1, 45),   # 2048 passages per wave, every XCD with a histogram of its own
    (300, 140_001, 2, 6, 13, 46),  # thirteen queries padded to sixteen
]


@pytest.mark.parametrize("C,P,lo,hi,nq,seed", CASES)
@pytest.mark.parametrize("stage2", ["inverted11", "inverted13"])
def test_pruned_stage2_keeps_the_best(C, P, lo, hi, nq, seed, stage2):
    import paper_2205_09707_amd as pl
    pl.load_library()
    w = make_workload(tiny_config(C=C, P=P, lo=lo, hi=hi, nq=nq, seed=seed), noise="calibrated")
    rowmax = np.sort(orc.scq(w.centroids.numpy(), w.queries[0].numpy()).max(axis=1))[::-1]
    params = []
    for K in (1, 2, 31, 40, 63, 64):  # survivors of the first query; the others have about as many
        t_cs = float((rowmax[K - 1] + rowmax[K]) / 2)
        params += [(2, t_cs, 16, 4), (4, t_cs, 1000, 50)]
    params.append((9, float(rowmax[20]), 300, 10))  # more probes than the kernel classifies
    tp._check_workload(pl, w, params, stage2=stage2, queries=sorted({0, nq // 2, nq - 1}))
