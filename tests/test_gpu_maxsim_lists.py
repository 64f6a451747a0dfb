"""Scores of long launches run over token lists packed across passages: passages of lengths around the groups of eight, the
steps of 32 and the chunks of 64 tokens, empty ones among them, against MaxSim in double on the decompressed vectors."""
import pytest
import torch

import parity_util as pu

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 2, 7, 8, 9, 15, 16, 17, 24, 31, 32, 33, 63, 64, 65, 72, 127, 128, 129, 191, 192, 193, 300, 700]
LONG = 48 * 768  # passages of a launch from which the lists are packed


def _index(pl, P, C, nbits, seed, lengths=LENGTHS):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    pick = torch.randint(0, len(lengths), (P,), generator=g, device="cuda")
    pick[:len(lengths)] = torch.arange(len(lengths), device="cuda")
    n = torch.tensor(lengths, device="cuda")[pick]
    offsets = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cumsum(n, 0)
    N = int(offsets[-1])
    cen = torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1)
    codes = (torch.rand(N, generator=g, device="cuda") ** 3 * C).int().clamp_(max=C - 1)
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, C)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.randint(0, 256, (N, 16 * nbits), generator=g, device="cuda", dtype=torch.uint8),
              "bucket_weights": torch.tensor([-0.09, -0.02, 0.03, 0.08][:1 << nbits] if nbits == 2 else [-0.05, 0.06], device="cuda")}
    return pl.plaid_index_from_view(arrays, nbits, device=0, copy=False), arrays, g


def _maxima(idx, pl, offsets, q, keep=None):
    """Sum over the query tokens of the largest dot product over each passage's tokens (those of keep), in double."""
    P = offsets.numel() - 1
    N = int(offsets[-1])
    vectors = pl.plaid_decompress_passages(idx, torch.arange(P, dtype=torch.int32, device="cuda"), N)[1][:N]
    dots = vectors.double() @ q.double().T
    if keep is not None:
        dots[~keep] = -float("inf")
    owner = torch.repeat_interleave(torch.arange(P, device="cuda"), offsets[1:] - offsets[:-1])
    best = torch.full((P, 32), -float("inf"), dtype=torch.float64, device="cuda")
    best.scatter_reduce_(0, owner[:, None].expand(-1, 32), dots, "amax")
    return best.sum(dim=1)


@pytest.mark.parametrize("nbits", [1, 2])
@pytest.mark.parametrize("renormalize", [False, True])
def test_final_scores_of_packed_lists(nbits, renormalize):
    import paper_2205_09707_amd as pl
    P, nq, n3 = 2000, 41, 900
    assert nq * n3 >= LONG
    idx, a, g = _index(pl, P, 600, nbits, 7 + nbits)
    try:
        if renormalize:
            pl.plaid_index_set_renormalize(idx, True)
        Q = torch.nn.functional.normalize(torch.randn(nq, 32, 128, generator=g, device="cuda"), dim=2).contiguous()
        ids, scores, b = pl.plaid_search_debug(idx, Q, 4, -1.0, 4 * n3, n3, want=["sel3_ids", "n3"])
        torch.cuda.synchronize()
        for q in range(0, nq, 5):
            ref = _maxima(idx, pl, a["doc_offsets"], Q[q])
            got = ids[q] >= 0
            n = int(b["n3"][q])
            assert 500 < n <= n3 and int(got.sum()) == n
            # every passage of the list once, the best first
            assert torch.equal(torch.sort(ids[q][got]).values, torch.sort(b["sel3_ids"][q, :n]).values)
            assert bool((scores[q][got][1:] <= scores[q][got][:-1]).all())
            assert float((scores[q][got].double() - ref[ids[q][got].long()]).abs().max()) < pu.TOL
    finally:
        pl.plaid_index_free(idx)


@pytest.mark.parametrize("nbits", [1, 2])
@pytest.mark.parametrize("C,nprobe", [(600, 4), (600, 1), (70_000, 300)])  # the last: more probe bits than LDS takes
def test_pruning_scores_and_final_scores_of_vanilla_lists(nbits, C, nprobe):
    import paper_2205_09707_amd as pl
    P, nq, ncand = 2601, 33, 1200
    assert nq * ncand >= LONG
    idx, a, g = _index(pl, P, C, nbits, 70 + nbits)
    try:
        Q = torch.nn.functional.normalize(torch.randn(nq, 32, 128, generator=g, device="cuda"), dim=2).contiguous()
        ids, scores, b = pl.plaid_search_vanilla(idx, Q, nprobe, ncand, ncand, debug=True)
        torch.cuda.synchronize()
        for q in range(0, nq, 8):
            S = a["centroids"].double() @ Q[q].double().T
            probed = torch.zeros(C, dtype=torch.bool, device="cuda")
            probed[torch.topk(S, nprobe, dim=0).indices.reshape(-1)] = True
            n_cand, n_kept = int(b["n_cand"][q]), int(b["n_kept"][q])
            kept = b["kept_ids"][q, :n_kept].long()
            ref = _maxima(idx, pl, a["doc_offsets"], Q[q], probed[a["codes"].long()])
            if n_cand > ncand:
                assert n_kept == ncand
                assert float((b["kept_scores"][q, :n_kept].double() - ref[kept]).abs().max()) < pu.TOL
                # nothing that was left out is better than the last one kept
                left = torch.ones(P, dtype=torch.bool, device="cuda")
                left[kept] = False
                assert float(ref[left].max()) < float(ref[kept].min()) + pu.TOL
            full = _maxima(idx, pl, a["doc_offsets"], Q[q])
            got = ids[q] >= 0
            assert torch.equal(torch.sort(ids[q][got].long()).values, torch.sort(kept).values)
            assert float((scores[q][got].double() - full[ids[q][got].long()]).abs().max()) < pu.TOL
    finally:
        pl.plaid_index_free(idx)
