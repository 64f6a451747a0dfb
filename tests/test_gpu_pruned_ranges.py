"""The inverted stage-2 kernel scores only the passages whose bound reaches the best ndocs scores seen so far: what it keeps
must be the oracle's ndocs best whatever the number of survivors (bit planes of 31, 36 and 63 slots, and beyond), of
passages (128- and 2048-passage steps, ragged ends, several steps per wave) and of queries (their order over the XCDs).
Small collections are compared with the oracle, those that fill the chip with the streaming form, which the oracle checks
elsewhere."""
import numpy as np
import pytest

from oracle import oracle as orc
from synth import make_workload, tiny_config

import test_gpu_even_cost as te
import test_gpu_parity as tp

pytestmark = pytest.mark.gpu

CASES = [
    # C, P, lo, hi, queries, seed: one or several ranges, ragged or not
    (400, 127, 1, 9, 1, 41),
    (400, 128, 1, 9, 7, 42),
    (400, 2049, 1, 9, 9, 43),
    (300, 8192, 2, 12, 8, 44),
    (300, 140_001, 2, 6, 1, 45),   # 2048 passages per wave
    (300, 140_001, 2, 6, 13, 46),  # thirteen queries spread over the XCDs, a histogram copy each
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


def _launch(P, nq):
    """The launch rules of k_stage2.hip for collections of more than 40 ranges of 2048 passages (and an ndocs far below P)."""
    ranges = -(-P // 2048)
    steps = 4 if nq * ranges >= 16 * 12288 else (2 if nq * ranges >= 4 * 12288 else 1)
    blocks = -(-P // (4 * steps * 2048))
    spread = nq <= 32
    nqx = nq | 1 if spread else (nq + 7) // 8 * 8
    return {"steps": steps, "copies": spread and nq * blocks > 64, "padded": not spread and nqx > nq,
            "one_instance": nq < 8 or blocks * nqx <= 768, "two_areas": blocks * nqx <= 768}


@pytest.mark.parametrize("P,nq,claims", [
    (600_001, 1, {"copies": True, "two_areas": True, "steps": 1}),
    (110_001, 5, {"copies": True, "two_areas": True}),
    (500_000, 7, {"copies": True, "two_areas": True}),
    (1_500_000, 7, {"copies": True, "two_areas": False, "one_instance": True}),
    (900_001, 9, {"copies": True, "one_instance": False, "steps": 1}),
    (100_000, 33, {"copies": False, "padded": True, "one_instance": True}),
    (200_000, 40, {"copies": False, "padded": False, "one_instance": False}),
    (200_001, 512, {"steps": 2}),
    (790_000, 512, {"steps": 4}),
])
@pytest.mark.parametrize("stage2", ["inverted11", "inverted13"])
def test_launches_that_fill_the_chip(monkeypatch, P, nq, claims, stage2):
    import torch

    import paper_2205_09707_amd as pl
    pl.load_library()
    shape = _launch(P, nq)
    assert {k: shape[k] for k in claims} == claims, shape
    inv, Q, cen = te._index(monkeypatch, pl, 2048, P, 5, P % 1000, stage2, centroids=True, nq=nq)
    stream, _ = te._index(monkeypatch, pl, 2048, P, 5, P % 1000, "stream", nq=nq)
    try:
        for K in (1, 31, 40, 63, 64):  # survivors of a middling query; the others have about as many
            t_cs = sorted(te._thresholds(cen, Q[:9], K))[min(4, nq // 2)]
            a, b = (pl.plaid_search(x, Q, 3, t_cs, 900, 60) for x in (inv, stream))
            assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]), (P, nq, K)
    finally:
        pl.plaid_index_free(inv)
        pl.plaid_index_free(stream)
