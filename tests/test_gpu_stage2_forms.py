"""The streaming form and both inverted forms return the same ids and scores for whatever they are asked: random collections
(empty and long passages, repeated centroids, even and skewed popularity), batch sizes around the launch rules, survivor
counts around the slot limits, few and many probes, ndocs from one passage to all of them and more."""
import random

import pytest
import torch

pytestmark = pytest.mark.gpu
INF = float("inf")


@pytest.mark.parametrize("seed", range(12))
def test_forms_agree(monkeypatch, seed):
    import paper_2205_09707_amd as pl
    pl.load_library()
    rng = random.Random(seed)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    C, P = int(2 ** rng.uniform(1, 15)), int(2 ** rng.uniform(0, 19))
    mean = min(rng.choice([1, 3, 10, 40]), max(1, (1 << 22) // P))
    skew, nbits = rng.choice([1.0, 2.0, 3.0]), rng.choice([1, 2])
    lengths = torch.randint(0, 2 * mean + 1, (P,), generator=g, device="cuda")
    lengths[P // 2] = 700
    offsets = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = lengths.cumsum(0)
    N = int(offsets[-1])
    cen = torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1)
    if seed % 4 == 0:  # every row about three times
        cen = cen[torch.randint(0, C // 3 + 1, (C,), generator=g, device="cuda")]
    cen = cen.contiguous()

    def popular(n):
        return (C * torch.rand(n, generator=g, device="cuda") ** skew).long().clamp_(max=C - 1)
    codes = popular(N).int()
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, C)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.randint(0, 256, (N, 16 * nbits), generator=g, device="cuda", dtype=torch.uint8),
              "bucket_weights": torch.linspace(-0.05, 0.05, 1 << nbits, device="cuda")}
    Q = cen[popular(64 * 32)] + 0.03 * torch.randn(64 * 32, 128, generator=g, device="cuda")
    Q = torch.nn.functional.normalize(Q, dim=1).reshape(64, 32, 128)
    if seed % 3 == 0:  # other norms: few survivors for some queries, many for others
        Q = Q * (0.3 + 1.5 * torch.rand(64, 1, 1, generator=g, device="cuda"))
    best = torch.sort((cen @ Q[0].T).max(1).values, descending=True).values
    index = {}
    for form in ("stream", "inverted11", "inverted13"):
        with monkeypatch.context() as mp:
            mp.setenv("PLAID_STAGE2_FORM", form)
            index[form] = pl.plaid_index_from_view(arrays, nbits, device=0, copy=False)
    try:
        for nq in (1, rng.choice([2, 7, 8]), rng.choice([9, 16, 31]), rng.choice([32, 33, 40]), 64):
            q = Q[:nq].contiguous()
            for _ in range(2):
                K = rng.choice([0, 1, 5, 20, 31, 32, 36, 37, 50, 63, 64, 65, 200, C])
                t_cs = float(best[min(K, C) - 1]) - 1e-6 if K else rng.choice([-INF, -2.0, INF, float(best[0]) + 0.01])
                nprobe = min(C, rng.choice([1, 2, 4, 8, 9, 40]))
                ndocs, k = min(rng.choice([1, 10, 256, 5000, P, 2 * P]), 20000), rng.choice([1, 10, 1000])
                case = f"C={C} P={P} N={N} nq={nq} K={K} t_cs={t_cs} nprobe={nprobe} ndocs={ndocs} k={k}"
                print(case, flush=True)
                want = pl.plaid_search(index["stream"], q, nprobe, t_cs, ndocs, k)
                for form in ("inverted11", "inverted13"):
                    got = pl.plaid_search(index[form], q, nprobe, t_cs, ndocs, k)
                    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), (form, case)
    finally:
        for idx in index.values():
            pl.plaid_index_free(idx)
