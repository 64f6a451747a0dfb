"""The ndocs cut of launches of few queries (and, beside them, of many): boundary lists longer than LDS holds whose keys differ in
their scores within the bin, in their ids alone, or in both, so that each kind of digit and the pass after it decide; lists that end
at a workgroup's step (4096 keys) and at what LDS holds (8192)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,near", [(8193, 50), (12_288, 1), (12_289, 2), (40_961, 50), (600_001, 50), (600_001, 3)])
@pytest.mark.parametrize("nq", [1, 32, 33])
def test_cuts_within_a_bin(P, near, nq):
    """`near` centroids score almost the same, far above one other survivor that stretches the bins: their passages, one token
    each, share a bin or two, with as many distinct scores as there are such centroids."""
    import paper_2205_09707_amd as pl
    g = torch.Generator(device="cuda")
    g.manual_seed(P + near)
    C = 64
    q = torch.nn.functional.normalize(torch.randn(128, generator=g, device="cuda"), dim=0)
    cen = torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1)
    cen[:near] = torch.nn.functional.normalize(q + 2e-3 * torch.randn(near, 128, generator=g, device="cuda"), dim=1)
    other = cen[near] - (cen[near] @ q) * q
    cen[near] = 0.3 * q + (1 - 0.09) ** 0.5 * other / other.norm()  # the survivor far below
    codes = torch.randint(0, near, (P,), generator=g, device="cuda", dtype=torch.int32)
    codes[::97] = near
    offsets = torch.arange(P + 1, dtype=torch.int64, device="cuda")
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, C)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.full((P, 32), 27, dtype=torch.uint8, device="cuda"),
              "bucket_weights": torch.tensor([-0.02, -0.01, 0.01, 0.02], device="cuda")}
    idx = pl.plaid_index_from_view(arrays, 2, device=0, copy=False)
    try:
        Q = q.expand(nq, 32, 128).contiguous()
        # 32 equal query tokens: a passage's score is 32 times its centroid's, whatever the rounding of one of them
        dot = (cen.double() @ q.double()).float()
        order = torch.argsort(dot[codes.long()], descending=True, stable=True)
        nprobe = min(C, 8)
        cand = torch.zeros(C, dtype=torch.bool, device="cuda")
        cand[torch.topk(dot, nprobe).indices] = True
        order = order[cand[codes.long()][order]]
        order = order[dot[codes.long()[order]] >= 0.25]
        n = len(order)
        for m in sorted({1, 4095, 4097, n // 3, n - 1}):
            if m < 1 or m > n:
                continue
            _, _, dbg = pl.plaid_search_debug(idx, Q, nprobe, 0.25, m, 1, want=["sel2_ids", "n2"])
            for i in {0, nq - 1}:
                assert int(dbg["n2"][i]) == m
                kept = torch.sort(dbg["sel2_ids"][i, :m].long()).values
                assert torch.equal(kept, torch.sort(order[:m]).values), (m, i)
    finally:
        pl.plaid_index_free(idx)


@pytest.mark.parametrize("P", [40_961, 600_001])
@pytest.mark.parametrize("near,apart", [(2, 1), (2, 16), (3, 400), (7, 170), (7, 171)])
def test_scores_closer_than_a_digit(P, near, apart):
    """`near` scores, `apart` representable numbers from one to the next and many passages each: up to 1023 between the first and the
    last they are told apart by their lowest bits, here so that these come round from 1023 to 0 between the first and the second."""
    import paper_2205_09707_amd as pl
    C = 64
    q = torch.zeros(128, device="cuda")
    q[0] = 1.0
    cen = torch.zeros(C, 128, device="cuda")
    # products with q are exact, and 32 of them lie in [16, 32), whose spacing is 2^-19: 1024 of those is a multiple of 2^-9
    cen[:near, 0] = 1.0 - 2.0 ** -14 + 2.0 ** -24 * (apart // 2) - 2.0 ** -24 * apart * torch.arange(near, device="cuda")
    cen[near, 0] = 0.3  # the survivor far below stretches the bins
    cen[near + 1:, 1] = 1.0
    codes = (torch.arange(P, device="cuda") * 7919 % 1009 % near).int()
    codes[::97] = near
    offsets = torch.arange(P + 1, dtype=torch.int64, device="cuda")
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, C)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.full((P, 32), 27, dtype=torch.uint8, device="cuda"),
              "bucket_weights": torch.tensor([-0.02, -0.01, 0.01, 0.02], device="cuda")}
    idx = pl.plaid_index_from_view(arrays, 2, device=0, copy=False)
    try:
        order = torch.argsort(codes, stable=True)  # the centroids' numbers fall with their scores
        per = int((codes == 0).sum())
        for nq in (1, 32):
            Q = q.expand(nq, 32, 128).contiguous()
            for m in (1, 5000, per - 1, per, per + 1, per + 5000, near * per - 3, P // 2, P - 1):
                _, _, dbg = pl.plaid_search_debug(idx, Q, 8, 0.25, m, 1, want=["sel2_ids", "n2"])
                for i in {0, nq - 1}:
                    assert int(dbg["n2"][i]) == m
                    kept = torch.sort(dbg["sel2_ids"][i, :m].long()).values
                    assert torch.equal(kept, torch.sort(order[:m]).values), (m, nq, i)
    finally:
        pl.plaid_index_free(idx)
