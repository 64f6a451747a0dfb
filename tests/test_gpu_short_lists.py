"""Short lists, few in all, are cut and scored by one launch, others by two: both give the same results, bit for bit.  Lists around one workgroup's
threads and the longest that the launch takes, more and fewer of them than it takes, repeated passages (ties at the cut), empty ones, queries
with fewer candidates than that.  And what the cut keeps and the time of the stages come from the launches of an ordinary search."""
import pytest
import torch

import test_gpu_maxsim_lists as lists

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbits,renormalize", [(1, False), (2, False), (1, True), (2, True)])
@pytest.mark.parametrize("nq,ndocs", [(1, 4), (3, 5), (2, 255), (32, 256), (33, 256), (7, 257), (1, 1023), (8, 1024), (9, 1024), (1, 1025)])
def test_cut_and_scores_in_one_launch(nbits, renormalize, nq, ndocs):
    import paper_2205_09707_amd as pl
    P, C = 4000, 400
    idx, a, g = lists._index(pl, P, C, nbits, 31 + nbits, lists.LENGTHS[:-1] if nq > 1 else lists.LENGTHS)
    try:
        if renormalize:
            pl.plaid_index_set_renormalize(idx, True)
        # (the codes of the first centroids are most frequent)
        Q = torch.nn.functional.normalize(a["centroids"][:nq, None] + 0.3 * torch.randn(nq, 32, 128, generator=g, device="cuda"), dim=2).contiguous()
        for k, t_cs in [(1, -1.0), (max(1, ndocs // 4), -1.0), (max(1, ndocs // 4), 0.9)]:
            ids, scores = pl.plaid_search(idx, Q, 2, t_cs, ndocs, k)
            want_ids, want_scores, b = pl.plaid_search_debug(idx, Q, 2, t_cs, ndocs, k, want=["sel3_ids", "n3", "sel3_scores"])
            torch.cuda.synchronize()
            assert int(b["n3"].max()) >= min(k, ndocs // 4)
            assert torch.equal(ids, want_ids) and torch.equal(scores, want_scores), (k, t_cs)
            # the same queries among so many that the cut has a launch of its own (not for so few keys a query: a chunk has 512 queries)
            if ndocs <= 16:
                continue
            many = Q[torch.arange(max(nq, 8192 // ndocs + 1), device="cuda") % nq].contiguous()
            two_ids, two_scores, c = pl.plaid_search_debug(idx, many, 2, t_cs, ndocs, k, want=["sel3_ids", "n3", "sel3_scores"])
            torch.cuda.synchronize()
            assert torch.equal(ids, two_ids[:nq]) and torch.equal(scores, two_scores[:nq]) and torch.equal(b["n3"], c["n3"][:nq]), (k, t_cs)
            for q in range(nq):
                n = int(b["n3"][q])
                (x, a1), (y, a2) = ((torch.sort(d["sel3_ids"][q, :n])) for d in (b, c))
                assert torch.equal(x, y) and torch.equal(b["sel3_scores"][q, :n][a1], c["sel3_scores"][q, :n][a2]), (k, t_cs, q)
    finally:
        pl.plaid_index_free(idx)


@pytest.mark.parametrize("nq,ndocs", [(1, 256), (12, 1024), (40, 300)])
def test_timing_and_what_the_cut_keeps_come_from_an_ordinary_searchs_kernels(nq, ndocs):
    import paper_2205_09707_amd as pl
    from torch.profiler import ProfilerActivity, profile
    idx, a, g = lists._index(pl, 4000, 400, 2, 5)
    try:
        Q = torch.nn.functional.normalize(a["centroids"][:nq, None] + 0.3 * torch.randn(nq, 32, 128, generator=g, device="cuda"), dim=2).contiguous()

        def kernels(call):
            call()
            torch.cuda.synchronize()
            with profile(activities=[ProfilerActivity.CUDA]) as p:
                call()
                torch.cuda.synchronize()
            names = [e.key for e in p.key_averages()]
            if not names:
                pytest.skip("no kernels from torch's profiler here")
            return sorted(n for n in names if any(k in n for k in ("stage1", "scq", "s2_", "sel", "ci_", "maxsim")))
        plain = kernels(lambda: pl.plaid_search(idx, Q, 2, 0.4, ndocs, 10))
        assert any("cut_maxsim" in n for n in plain) == (ndocs * nq <= 8192), plain
        asked = kernels(lambda: pl.plaid_search_debug(idx, Q, 2, 0.4, ndocs, 10, want=["sel3_ids", "sel3_scores", "n3"]))
        pl.plaid_set_stage_timing(idx, True)
        timed = kernels(lambda: pl.plaid_search(idx, Q, 2, 0.4, ndocs, 10))
        ms = list(pl.plaid_get_stage_ms(idx).values())
        pl.plaid_set_stage_timing(idx, False)
        assert asked == plain and timed == plain, (plain, asked, timed)
        if ndocs * nq <= 8192:
            assert ms[7] < ms[8], ms  # nothing, but for the time between two events
    finally:
        pl.plaid_index_free(idx)


def test_ties_at_the_cut():
    import paper_2205_09707_amd as pl
    C = 40
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    cen = torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1)
    codes = torch.randint(0, C, (30 * 5,), generator=g, device="cuda").int().repeat(40)  # thirty passages, forty times each
    offsets = 5 * torch.arange(1201, device="cuda")
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, C)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.randint(0, 256, (len(codes), 32), generator=g, device="cuda", dtype=torch.uint8),
              "bucket_weights": torch.linspace(-0.05, 0.05, 4, device="cuda")}
    idx = pl.plaid_index_from_view(arrays, 2, device=0, copy=False)
    try:
        Q = torch.nn.functional.normalize(torch.randn(4, 32, 128, generator=g, device="cuda"), dim=2).contiguous()
        for ndocs in (100, 640, 1024):
            ids, scores = pl.plaid_search(idx, Q, 4, -1.0, ndocs, ndocs // 4)
            want_ids, want_scores, b = pl.plaid_search_debug(idx, Q, 4, -1.0, ndocs, ndocs // 4, want=["sel3_ids", "n3"])
            torch.cuda.synchronize()
            assert int(b["n3"].min()) == ndocs // 4
            assert torch.equal(ids, want_ids) and torch.equal(scores, want_scores), ndocs
            many = Q[torch.arange(8192 // ndocs + 4, device="cuda") % 4].contiguous()  # the cut has a launch of its own
            two_ids, two_scores, c = pl.plaid_search_debug(idx, many, 4, -1.0, ndocs, ndocs // 4, want=["sel3_ids", "n3"])
            assert torch.equal(ids, two_ids[:4]) and torch.equal(scores, two_scores[:4]), ndocs
            assert torch.equal(torch.sort(b["sel3_ids"], dim=1).values, torch.sort(c["sel3_ids"][:4], dim=1).values), ndocs
    finally:
        pl.plaid_index_free(idx)
