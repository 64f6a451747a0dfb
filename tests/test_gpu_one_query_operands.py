"""A launch of one query forms its operands in the score kernel and clears the workspace there, unless that is too much for the
workgroups it has: either way its scores are, bit for bit, those the query gets in a launch of two."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,P,taken", [(64, 2000, False), (1024, 5000, True), (1000, 700_000, False), (20_001, 70_000, True)])
def test_one_query_scores_as_in_a_launch_of_two(C, P, taken):
    import paper_2205_09707_amd as pl
    g = torch.Generator(device="cuda")
    g.manual_seed(C + P)
    cen = torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1).contiguous()
    offsets = torch.arange(P + 1, dtype=torch.int64, device="cuda") * 3
    codes = torch.randint(0, C, (3 * P,), generator=g, device="cuda", dtype=torch.int32)
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, C)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.randint(0, 256, (3 * P, 32), generator=g, device="cuda", dtype=torch.uint8),
              "bucket_weights": torch.tensor([-0.05, -0.015, 0.015, 0.05], device="cuda")}
    # workspace words that start at zero: the candidate bitmap, three histograms, the selections' state
    words = (P + 31) // 32 + 3 * 2048 + 2 * (16 + 2 * 2048)
    assert (words <= 32 * 256 * ((C + 255) // 256)) == taken
    idx = pl.plaid_index_from_view(arrays, 2, device=0, copy=False)
    try:
        Q = torch.nn.functional.normalize(cen[codes[:64].long()].reshape(2, 32, 128) + 0.03 * torch.randn(2, 32, 128, generator=g, device="cuda"), dim=2)
        two_ids, two_scores, two = pl.plaid_search_debug(idx, Q.contiguous(), 2, 0.4, 200, 10, want=["S_cq", "keep", "probed"])
        for i in range(2):
            for _ in range(2):  # (the second time over what the first one left in the workspace)
                ids, scores, one = pl.plaid_search_debug(idx, Q[i:i + 1].contiguous(), 2, 0.4, 200, 10, want=["S_cq", "keep", "probed"])
                for name in ("S_cq", "keep", "probed"):
                    assert torch.equal(one[name][0], two[name][i]), name
                assert torch.equal(ids[0], two_ids[i]) and torch.equal(scores[0], two_scores[i])
    finally:
        pl.plaid_index_free(idx)
