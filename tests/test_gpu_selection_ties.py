"""The ndocs cut through one or two groups of equal scores, of lengths around the keys a workgroup takes per step of the filters
(2048) and the list lengths from which the digit filters run: ties go to the smaller passage ids."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [1, 63, 2047, 2048, 2049, 4096, 4097, 8193, 40_961, 600_001])
@pytest.mark.parametrize("nq", [1, 9, 40])
def test_cuts_through_equal_scores(P, nq):
    import paper_2205_09707_amd as pl
    g = torch.Generator(device="cuda")
    g.manual_seed(P)
    cen = torch.nn.functional.normalize(torch.randn(64, 128, generator=g, device="cuda"), dim=1)
    # one token per passage: every third lies at centroid 0 (the best score), the others at centroid 1
    codes = (torch.arange(P, device="cuda") % 3 != 0).int()
    offsets = torch.arange(P + 1, dtype=torch.int64, device="cuda")
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, 64)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.full((P, 32), 27, dtype=torch.uint8, device="cuda"),
              "bucket_weights": torch.tensor([-0.02, -0.01, 0.01, 0.02], device="cuda")}
    idx = pl.plaid_index_from_view(arrays, 2, device=0, copy=False)
    try:
        q = torch.nn.functional.normalize(1.0 * cen[0] + 0.6 * cen[1], dim=0)
        Q = q.expand(nq, 32, 128).contiguous()
        first = torch.arange(0, P, 3, device="cuda")
        order = torch.cat([first, torch.tensor([p for p in range(min(P, 40_000)) if p % 3], dtype=torch.int64, device="cuda")])
        for m in sorted({1, 5, min(P, 2048), min(P, len(first) + 1), min(P, len(first) + 700), min(P, 9000)}):
            if m > len(order):
                continue
            k = max(1, m // 4)
            _, _, dbg = pl.plaid_search_debug(idx, Q, 2, 0.1, m, k, want=["sel2_ids", "n2"])
            for i in {0, nq // 2, nq - 1}:
                assert int(dbg["n2"][i]) == m
                kept = torch.sort(dbg["sel2_ids"][i, :m].long()).values
                assert torch.equal(kept, torch.sort(order[:m]).values), (m, i)
    finally:
        pl.plaid_index_free(idx)


@pytest.mark.parametrize("P,step", [(1000, 3), (32_769, 5), (300_000, 1), (600_001, 97), (600_001, 7)])
def test_candidates_without_a_surviving_centroid_fill_in_id_order(P, step):
    """The first bitmap words one per thread, then eight, the last slots one again: whole rounds, the round of the cut and an
    end of the bitmap before the slots are full."""
    import paper_2205_09707_amd as pl
    g = torch.Generator(device="cuda")
    g.manual_seed(P + step)
    cen = torch.nn.functional.normalize(torch.randn(64, 128, generator=g, device="cuda"), dim=1)
    codes = (torch.arange(P, device="cuda") % step != 0).int() * 9  # every step-th passage lies at centroid 0
    offsets = torch.arange(P + 1, dtype=torch.int64, device="cuda")
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, 64)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.full((P, 32), 27, dtype=torch.uint8, device="cuda"),
              "bucket_weights": torch.tensor([-0.02, -0.01, 0.01, 0.02], device="cuda")}
    idx = pl.plaid_index_from_view(arrays, 2, device=0, copy=False)
    try:
        Q = cen[0].expand(2, 32, 128).contiguous()
        cand = torch.arange(0, P, step, device="cuda")
        for m in (1, 300, 3000, 6500):
            _, _, dbg = pl.plaid_search_debug(idx, Q, 1, 5.0, m, 10, want=["sel2_ids", "n2"])
            n = min(m, len(cand))
            for i in range(2):
                assert int(dbg["n2"][i]) == n
                assert torch.equal(torch.sort(dbg["sel2_ids"][i, :n].long()).values, cand[:n]), m
    finally:
        pl.plaid_index_free(idx)
