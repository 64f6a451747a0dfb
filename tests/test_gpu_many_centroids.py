"""More than 2^25 centroids: a row of S_cq then lies up to C * 128 bytes = more than 2^32 into a query's scores.  The final scores
of every form of stage 4 (a workgroup per passage, a wave per passage, packed lists; lists that are cut by the same launch) against MaxSim in
double on the decompressed vectors; the tokens lie at the last centroids and at those whose rows 32-bit offsets would reach in their place."""
import pytest
import torch

import parity_util as pu
from test_gpu_maxsim_lists import LONG, _maxima

pytestmark = pytest.mark.gpu


def _arrays(pl, nbits):
    C, P = (1 << 25) + 40, 8000
    g = torch.Generator(device="cuda")
    g.manual_seed(25)
    cen = torch.empty(C, 128, device="cuda")
    for c0 in range(0, C, 1 << 22):  # (one piece at a time: 17 GB in all)
        n = min(1 << 22, C - c0)
        cen[c0:c0 + n] = torch.nn.functional.normalize(torch.randn(n, 128, generator=g, device="cuda"), dim=1)
    offsets = torch.arange(P + 1, dtype=torch.int64, device="cuda") * 5
    codes = torch.randint(0, 40, (5 * P,), generator=g, device="cuda")
    codes = torch.where(torch.rand(5 * P, generator=g, device="cuda") < 0.7, codes + (1 << 25), codes).int()
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, C)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.randint(0, 256, (5 * P, 16 * nbits), generator=g, device="cuda", dtype=torch.uint8),
              "bucket_weights": torch.tensor([-0.09, -0.02, 0.03, 0.08][-1 << nbits:], device="cuda")}
    src = codes[torch.randint(0, 5 * P, (5 * 32,), generator=g, device="cuda")].long()
    Q = cen[src] + 0.02 * torch.randn(5 * 32, 128, generator=g, device="cuda")
    return arrays, torch.nn.functional.normalize(Q, dim=1).reshape(5, 32, 128).contiguous()


def test_final_scores_with_rows_past_32_bit_offsets():
    import paper_2205_09707_amd as pl
    pl.load_library()
    nbits = 2
    arrays, Q = _arrays(pl, nbits)
    offsets, P = arrays["doc_offsets"], arrays["doc_offsets"].numel() - 1
    idx = pl.plaid_index_from_view(arrays, nbits, device=0, copy=False)
    try:
        ref = [_maxima(idx, pl, offsets, Q[q]) for q in range(5)]
        for nq, ndocs in ((1, 2000), (5, 2000), (5, 4 * P)):
            n3 = min(P, ndocs // 4)
            assert (nq * n3 > 2048) == (nq > 1) and (nq * n3 >= LONG) == (ndocs > P)
            ids, scores = pl.plaid_search(idx, Q[:nq], 4, 0.3, ndocs, n3)
            torch.cuda.synchronize()
            for q in range(nq):
                got = ids[q] >= 0
                assert int(got.sum()) >= n3 // 2
                worst = float((scores[q][got].double() - ref[q][ids[q][got].long()]).abs().max())
                assert worst < pu.TOL, (nq, ndocs, q)
    finally:
        pl.plaid_index_free(idx)


@pytest.mark.parametrize("nbits", [1, 2])
def test_final_scores_of_short_lists_with_rows_past_32_bit_offsets(nbits):
    import paper_2205_09707_amd as pl
    pl.load_library()
    arrays, Q = _arrays(pl, nbits)
    offsets = arrays["doc_offsets"]
    idx = pl.plaid_index_from_view(arrays, nbits, device=0, copy=False)
    try:
        for renormalize in (False, True):
            pl.plaid_index_set_renormalize(idx, renormalize)
            for nq, ndocs in ((1, 1000), (1, 1024), (5, 100)):
                ids, scores = pl.plaid_search(idx, Q[:nq], 4, 0.3, ndocs, ndocs // 4)
                torch.cuda.synchronize()
                for q in range(nq):
                    ref = _maxima(idx, pl, offsets, Q[q])
                    assert bool((ids[q] >= 0).all())
                    assert float((scores[q].double() - ref[ids[q].long()]).abs().max()) < pu.TOL, (renormalize, nq, ndocs, q)
    finally:
        pl.plaid_index_free(idx)
