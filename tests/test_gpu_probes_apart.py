"""Launches of fewer than 32 queries find a query's probes by a workgroup per eight of its tokens and leave the duplicates among them to
stage 2; larger ones by one workgroup, which forms the union.  Both give the same probes, candidates and results: around the smallest
tables that are split, with duplicates throughout (few centroids), with more rows per token than a workgroup stages (repeated rows) and with
groups of tiles."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,copies,nprobe", [(31, 1, 1), (32, 1, 1), (64, 1, 2), (63, 1, 2), (256, 1, 8), (255, 1, 8), (700, 1, 3), (2100, 5, 4),
                                             (6000, 40, 2), (9000, 1, 5), (34_000, 3, 4)])
def test_queries_in_one_launch_and_a_few_at_a_time(C, copies, nprobe):
    import paper_2205_09707_amd as pl
    pl.load_library()
    P, nq = 3000, 33
    g = torch.Generator(device="cuda")
    g.manual_seed(C + nprobe)
    cen = torch.nn.functional.normalize(torch.randn(-(-C // copies), 128, generator=g, device="cuda"), dim=1)
    cen = cen.repeat_interleave(copies, dim=0)[:C].contiguous()
    offsets = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cumsum(torch.randint(0, 12, (P,), generator=g, device="cuda"), 0)
    N = int(offsets[-1])
    codes = (torch.rand(N, generator=g, device="cuda") ** 3 * C).int().clamp_(max=C - 1)  # some in most passages
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, C)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.randint(0, 256, (N, 32), generator=g, device="cuda", dtype=torch.uint8),
              "bucket_weights": torch.linspace(-0.05, 0.05, 4, device="cuda")}
    # tokens around few centroids: the same probes many times over
    src = codes[torch.randint(0, N, (nq * 32,), generator=g, device="cuda")].long()
    Q = torch.nn.functional.normalize(cen[src] + 0.03 * torch.randn(nq * 32, 128, generator=g, device="cuda"), dim=1)
    Q = Q.reshape(nq, 32, 128).contiguous()
    idx = pl.plaid_index_from_view(arrays, 2, device=0, copy=False)
    try:
        got = {}
        for chunk in (nq, 31, 8, 1):
            pl.plaid_set_max_chunk(idx, chunk)
            got[chunk] = [(pl.plaid_search_debug(idx, Q, nprobe, t_cs, 400, 50, want=["probed", "cand", "n_cand"]),
                           pl.plaid_search(idx, Q, nprobe, t_cs, 400, 50)) for t_cs in (0.5, 0.3)]
        torch.cuda.synchronize()
        for chunk in (31, 8, 1):
            for (a, b), (x, y) in zip(got[nq], got[chunk]):
                assert torch.equal(a[2]["probed"], x[2]["probed"]) and torch.equal(a[2]["n_cand"], x[2]["n_cand"]), chunk
                for q in range(nq):
                    n = int(a[2]["n_cand"][q])
                    assert torch.equal(a[2]["cand"][q, :n], x[2]["cand"][q, :n]), (chunk, q)
                assert torch.equal(b[0], y[0]) and torch.equal(b[1], y[1]) and torch.equal(a[0], x[0]) and torch.equal(a[1], x[1]), chunk
    finally:
        pl.plaid_index_free(idx)


@pytest.mark.parametrize("P,nprobe,nq", [(900, 1, 34), (70_001, 4, 40), (70_001, 8, 33)])
def test_queries_of_the_gather_form_in_one_launch_and_a_few_at_a_time(P, nprobe, nq):
    """Queries with more surviving centroids than there are slots (S2_MAX_KEPT, 63) take their candidates from the probes in workgroups of
    their own, which drop the duplicates too: all tokens of a query at four centroids, one of them in most passages (its list has a bitmap)."""
    import paper_2205_09707_amd as pl
    pl.load_library()
    C = 3000
    g = torch.Generator(device="cuda")
    g.manual_seed(P + nprobe)
    cen = torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1)
    offsets = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cumsum(torch.randint(0, 12, (P,), generator=g, device="cuda"), 0)
    N = int(offsets[-1])
    codes = (torch.rand(N, generator=g, device="cuda") ** 6 * C).int().clamp_(max=C - 1)
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, C)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.randint(0, 256, (N, 32), generator=g, device="cuda", dtype=torch.uint8),
              "bucket_weights": torch.linspace(-0.05, 0.05, 4, device="cuda")}
    src = torch.randint(0, C, (nq, 4), generator=g, device="cuda")
    src[:, 0] = 0
    Q = torch.nn.functional.normalize(cen[src.repeat(1, 8)] + 0.02 * torch.randn(nq, 32, 128, generator=g, device="cuda"), dim=2).contiguous()
    idx = pl.plaid_index_from_view(arrays, 2, device=0, copy=False)
    try:
        got = {}
        for chunk in (nq, 31, 9, 8, 1):
            pl.plaid_set_max_chunk(idx, chunk)
            got[chunk] = (pl.plaid_search_debug(idx, Q, nprobe, 0.15, 400, 50, want=["probed", "cand", "n_cand", "keep"]),
                          pl.plaid_search(idx, Q, nprobe, 0.15, 400, 50))
        torch.cuda.synchronize()
        a, b = got[nq]
        survivors = sum((a[2]["keep"] >> s & 1).sum(1) for s in range(32))
        assert int(survivors.min()) > 63
        assert all(len(torch.unique(a[2]["probed"][q])) < 32 * nprobe for q in range(nq))
        for chunk in (31, 9, 8, 1):
            x, y = got[chunk]
            assert torch.equal(a[2]["probed"], x[2]["probed"]) and torch.equal(a[2]["n_cand"], x[2]["n_cand"]), chunk
            for q in range(nq):
                n = int(a[2]["n_cand"][q])
                assert torch.equal(a[2]["cand"][q, :n], x[2]["cand"][q, :n]), (chunk, q)
            assert torch.equal(b[0], y[0]) and torch.equal(b[1], y[1]) and torch.equal(a[0], x[0]) and torch.equal(a[1], x[1]), chunk
    finally:
        pl.plaid_index_free(idx)
