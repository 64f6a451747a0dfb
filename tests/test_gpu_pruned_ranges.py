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
    steps = 4 if nq * ranges >= 16 * 12288 else (2 if nq * ranges >= 4 * 12288 or (nq == 1 and 4096 < ranges <= 7000) else 1)
    blocks = -(-P // (4 * steps * 2048))
    spread = nq <= 32
    nqx = nq | 1 if spread else (nq + 7) // 8 * 8
    return {"steps": steps, "copies": spread and nq * blocks > 64, "padded": not spread and nqx > nq,
            "one_instance": nq < 8 or blocks * nqx <= 768, "two_areas": blocks * nqx <= 768,
            "four_areas": 4 * blocks * nqx <= 1024, "tall_alone": 1024 < 2 * blocks * nqx <= 1536}


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


def _uneven_columns(monkeypatch, pl, P, nq, forms):
    """Passages of five tokens, each 2048 of them with tokens of another number (0 to 63) and choice of the first 63 centroids, and
    nq queries whose token i lies between centroids 2 i and 2 i + 1: at a threshold of 0.55 those 63 survive, and the planes that
    a range needs are as many as its column holds."""
    import torch
    C, length = 4096, 5
    g = torch.Generator(device="cuda")
    g.manual_seed(P)
    cen = torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1).contiguous()
    codes = torch.randint(64, C, (P, length), generator=g, device="cuda", dtype=torch.int32)
    col = torch.arange(-(-P // 2048), device="cuda").repeat_interleave(63 * 2)
    s = torch.arange(63, device="cuda").repeat_interleave(2).repeat(-(-P // 2048))
    n = 7 * col % 64
    at = col * 2048 + torch.randint(0, 2048, (col.numel(),), generator=g, device="cuda")
    use = (s < n) & (at < P)
    codes[at[use], s[use] % length] = ((5 * s + col) % 63).int()[use]
    offsets = torch.arange(P + 1, device="cuda", dtype=torch.int64) * length
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes.reshape(-1), offsets, C)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes.reshape(-1), "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.randint(0, 256, (P * length, 32), generator=g, device="cuda", dtype=torch.uint8),
              "bucket_weights": torch.tensor([-0.05, -0.015, 0.015, 0.05], device="cuda")}
    i = torch.arange(32, device="cuda")
    near = cen[2 * i] + cen[(2 * i + 1).clamp_(max=62)]
    Q = near / near.norm(dim=1, keepdim=True) + 0.01 * torch.randn(nq, 32, 128, generator=g, device="cuda")
    Q[1::3, 20:] = Q[1::3, :12]  # every third query: tokens repeat, 40 survivors
    Q = torch.nn.functional.normalize(Q, dim=2).contiguous()
    index = []
    for form in forms:
        with monkeypatch.context() as mp:
            mp.setenv("PLAID_STAGE2_FORM", form)
            index.append(pl.plaid_index_from_view(arrays, 2, device=0, copy=False))
    return index, Q, cen


@pytest.mark.parametrize("P,nq,claims", [
    (100_001, 1, {"four_areas": True, "steps": 1}),
    (400_000, 5, {"four_areas": True, "steps": 1}),
    (600_001, 5, {"four_areas": False, "two_areas": True, "steps": 1}),
    (500_000, 11, {"two_areas": True, "tall_alone": True}),
    (8_600_000, 1, {"four_areas": False, "two_areas": True, "steps": 2}),
    (900_001, 9, {"one_instance": False, "steps": 1}),
    (200_001, 512, {"one_instance": False, "steps": 2}),
])
def test_ranges_whose_planes_do_not_fit(monkeypatch, P, nq, claims):
    """63 and 40 survivors without bitmaps: ranges whose columns hold more of them than a wave's area has planes for (26 or 24, twice or
    four times that where it has the areas of others) go in halves or quarters, their neighbours whole, one or two ranges per wave.
    Nine columns in ten hold a given list, so that with columns of 2048 passages and many workgroups the 63 go to the
    instance of 36 planes and the 40 do not (launches of some workgroups run that instance alone, also for queries of more than 63)."""
    import torch

    import paper_2205_09707_amd as pl
    pl.load_library()
    shape = _launch(P, nq)
    assert {k: shape[k] for k in claims} == claims, shape
    forms = ("stream", "inverted11", "inverted13")
    index, Q, cen = _uneven_columns(monkeypatch, pl, P, nq, forms)
    try:
        for q in range(min(nq, 3)):
            assert int(((cen @ Q[q].T).max(1).values >= 0.55).sum()) == (40 if q % 3 == 1 else 63)
        for nprobe, t_cs, ndocs in ((3, 0.55, 900), (2, 0.55, 100), (2, 0.3, 900)):
            want = pl.plaid_search(index[0], Q, nprobe, t_cs, ndocs, ndocs // 4)
            for form, idx in zip(forms[1:], index[1:]):
                got = pl.plaid_search(idx, Q, nprobe, t_cs, ndocs, ndocs // 4)
                assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), (form, nprobe, t_cs, ndocs)
    finally:
        for idx in index:
            pl.plaid_index_free(idx)
