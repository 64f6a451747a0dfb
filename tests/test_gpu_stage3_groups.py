"""Stage 3 takes a passage per wave in launches of at most 16384 of them, else two: scores on both sides of the line, and of lists that do not
fill their last workgroup, against the definition in double on the dumped S_cq."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,ndocs", [(1, 4), (1, 5), (3, 1021), (16, 1024), (17, 964), (33, 511)])
def test_scores_of_short_and_long_launches(nq, ndocs):
    import paper_2205_09707_amd as pl
    import test_gpu_maxsim_lists as lists
    idx, a, g = lists._index(pl, 2500, 600, 2, nq + ndocs, lengths=[0, 1, 7, 8, 9, 63, 64, 65, 128, 129, 200])
    try:
        Q = torch.nn.functional.normalize(torch.randn(nq, 32, 128, generator=g, device="cuda"), dim=2).contiguous()
        _, _, b = pl.plaid_search_debug(idx, Q, 4, -1.0, ndocs, 10, want=["S_cq", "sel3_ids", "sel3_scores", "n3"])
        torch.cuda.synchronize()
        codes, off = a["codes"].long(), a["doc_offsets"].tolist()
        for q in (0, nq // 2, nq - 1):
            n = int(b["n3"][q])
            for j in {0, 1, n // 2, n - 2, n - 1} & set(range(n)):
                p = int(b["sel3_ids"][q, j])
                rows = b["S_cq"][q][codes[off[p]:off[p + 1]]]
                want = rows.max(dim=0).values.double().sum().float() if len(rows) else torch.tensor(-float("inf"))
                assert float(b["sel3_scores"][q, j]) == pytest.approx(float(want), rel=2.0 ** -23), (q, j, p)  # (one rounding to fp32 each)
    finally:
        pl.plaid_index_free(idx)
