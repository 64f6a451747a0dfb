"""Vanilla retrieval that prunes by coarse scores first keeps and gives what pruning by full scores keeps and gives (the debug form that
returns the kept scores prunes by full ones): many and few candidates, ties at the cut, both code widths, chunks, residual weights below
fp16's range.  Which of the calls here prune coarsely is checked by test_build_properties.py."""
import ctypes as ct

import pytest
import torch

pytestmark = pytest.mark.gpu


def _index(pl, P, C, nbits, scale, copies, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    cen = torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1).contiguous()
    lengths = torch.randint(0, 30, (P // copies,), generator=g, device="cuda").repeat(copies)
    offsets = torch.zeros(len(lengths) + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cumsum(lengths, 0)
    N = int(offsets[-1])
    per = N // copies
    u = torch.rand(per, generator=g, device="cuda")
    codes = ((C - 1) * u ** 3).int().repeat(copies)  # some centroids in most passages
    res = torch.randint(0, 256, (per, 16 * nbits), generator=g, device="cuda", dtype=torch.uint8).repeat(copies, 1)
    io, ip = pl.plaid_build_ivf(codes, offsets, C)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": io, "ivf_pids": ip, "residuals": res,
              "bucket_weights": scale * torch.tensor([-1.5, -0.4, 0.4, 1.5][:1 << nbits] if nbits == 2 else [-0.9, 1.0], device="cuda")}
    idx = pl.plaid_index_from_view(arrays, nbits, device=0, copy=False)
    src = torch.randint(0, N, (16 * 32,), generator=g, device="cuda")
    Q = cen[codes[src].long()] + 0.03 * torch.randn(16 * 32, 128, generator=g, device="cuda")
    return idx, torch.nn.functional.normalize(Q, dim=1).reshape(16, 32, 128).contiguous(), arrays


def _kept(pl, idx, Q, nprobe, ncand, k):
    """What the call keeps when its scores are not asked for, as a plain call does."""
    nq = len(Q)
    b = {"ids": (nq, k), "cand": (nq, idx.P), "n_cand": (nq,), "kept_ids": (nq, ncand), "n_kept": (nq,)}
    b = {n: torch.zeros(shape, dtype=torch.int32, device="cuda") for n, shape in b.items()}
    b["scores"] = torch.zeros((nq, k), device="cuda")
    dbg = pl.plaid.plaid_vanilla_debug(**{n: b[n].data_ptr() for n in ("cand", "n_cand", "kept_ids", "n_kept")})
    rc = pl.load_library().plaid_search_vanilla(idx.handle, ct.c_void_p(Q.data_ptr()), nq, nprobe, ncand, k, ct.c_void_p(b["ids"].data_ptr()),
                                                ct.c_void_p(b["scores"].data_ptr()),
                                                ct.c_void_p(torch.cuda.current_stream().cuda_stream), ct.byref(dbg))
    assert rc == 0, pl.plaid_last_error()
    return b


@pytest.mark.parametrize("P,C,nbits,scale,copies,nprobe,ncand,chunk", [
    (70_000, 2048, 2, 0.02, 1, 4, 2000, None),
    (70_000, 2048, 1, 0.02, 1, 2, 17_000, None),
    (66_000, 1000, 2, 0.02, 3, 1, 1, None),        # every passage three times: ties at the cut
    (140_000, 1000, 2, 0.1, 4, 3, 4096, 6),        # ... in chunks of 6, 6 and 4, the last of which falls below the rule
    (200_000, 1000, 1, 0.1, 4, 3, 3000, 6),        # ... none does
    (70_000, 512, 2, 1e-5, 1, 1, 300, None),       # weights that fp16 cannot hold: the coarse scores miss the residuals
    (140_001, 70_000, 2, 0.02, 1, 1, 9000, None),  # some queries have no more candidates than that
])
def test_coarse_pruning_keeps_what_full_scores_keep(P, C, nbits, scale, copies, nprobe, ncand, chunk):
    import paper_2205_09707_amd as pl
    idx, Q, arrays = _index(pl, P, C, nbits, scale, copies, P + C)
    try:
        if chunk:
            pl.plaid_set_max_chunk(idx, chunk)
        k = min(ncand, 500)
        ids, scores = pl.plaid_search_vanilla(idx, Q, nprobe, ncand, k)
        want_ids, want_scores, dbg = pl.plaid_search_vanilla(idx, Q, nprobe, ncand, k, debug=True)
        got = _kept(pl, idx, Q, nprobe, ncand, k)
        torch.cuda.synchronize()
        print("candidates", dbg["n_cand"].tolist())
        assert torch.equal(ids, want_ids) and torch.equal(scores, want_scores)
        assert torch.equal(got["ids"], want_ids) and torch.equal(got["scores"], want_scores)
        assert torch.equal(got["n_cand"], dbg["n_cand"]) and torch.equal(got["n_kept"], dbg["n_kept"])
        assert bool((dbg["n_cand"] > ncand).any())  # (something is pruned)
        for q in range(len(Q)):
            n = int(dbg["n_kept"][q])
            assert n == min(ncand, int(dbg["n_cand"][q]))
            assert torch.equal(got["cand"][q, :int(got["n_cand"][q])], dbg["cand"][q, :int(got["n_cand"][q])])
            assert torch.equal(torch.sort(got["kept_ids"][q, :n]).values, torch.sort(dbg["kept_ids"][q, :n]).values), q
    finally:
        pl.plaid_index_free(idx)


def test_coarse_scores_decide_most_candidates():
    """The full scores of the few that they leave open take less time than the coarse scores of all."""
    import paper_2205_09707_amd as pl
    from torch.profiler import ProfilerActivity, profile
    idx, Q, _ = _index(pl, 200_000, 2048, 2, 0.02, 1, 9)
    try:
        pl.plaid_search_vanilla(idx, Q, 4, 2000, 100)
        torch.cuda.synchronize()
        with profile(activities=[ProfilerActivity.CUDA]) as p:
            pl.plaid_search_vanilla(idx, Q, 4, 2000, 100)
            torch.cuda.synchronize()
        us = {e.key: e.device_time_total for e in p.key_averages()}
        if not us:
            pytest.skip("no kernel times from torch's profiler here")
        coarse = sum(t for name, t in us.items() if "van_coarse_kernel" in name)
        full = sum(t for name, t in us.items() if "maxsim_list_kernel<2, true" in name)
        assert 0 < full < 0.5 * coarse
    finally:
        pl.plaid_index_free(idx)


@pytest.mark.parametrize("exponent", [-60, -36, -35, -34, -26, -16, -12, 0])
def test_queries_below_the_range_of_the_trailing_terms(exponent):
    """One passage leads by its centroid what its residual costs it.  Where the components are near 2^-36 the residual's part of the full
    score, formed of trailing terms below fp16's normal range, is up to twice the exact one, and the coarse score has none of it."""
    import paper_2205_09707_amd as pl
    P, w, ncand = 131_072, 0.0625, 64
    x = 1.02 * 2.0 ** exponent
    trailing = 2.0 ** -35 * round(x * 2 ** 35) / x if exponent <= -25 else 1.0  # of one: trailing term over exact value
    cen = torch.full((4, 128), -0.25, device="cuda")
    cen[0] = 0.25
    cen[1] = 0.25 + 2.3 * w / max(trailing, 1.0)
    codes = torch.zeros(P, dtype=torch.int32, device="cuda")
    codes[-1] = 1
    offsets = torch.arange(P + 1, dtype=torch.int64, device="cuda")
    io, ip = pl.plaid_build_ivf(codes, offsets, 4)
    res = torch.full((P, 16), 255, dtype=torch.uint8, device="cuda")
    res[-1] = 0
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": io, "ivf_pids": ip, "residuals": res,
              "bucket_weights": torch.tensor([-w, w], device="cuda")}
    idx = pl.plaid_index_from_view(arrays, 1, device=0, copy=False)
    try:
        Q = torch.full((8, 32, 128), x, device="cuda")
        ids, scores = pl.plaid_search_vanilla(idx, Q, 2, ncand, ncand)
        want_ids, want_scores, _ = pl.plaid_search_vanilla(idx, Q, 2, ncand, ncand, debug=True)
        torch.cuda.synchronize()
        assert torch.equal(ids, want_ids) and torch.equal(scores, want_scores)
    finally:
        pl.plaid_index_free(idx)


def test_queries_that_are_not_numbers():
    import paper_2205_09707_amd as pl
    idx, Q, arrays = _index(pl, 70_000, 2048, 2, 0.02, 1, 5)
    try:
        ids, scores = pl.plaid_search_vanilla(idx, Q, 2, 2000, 100)
        bad = Q.clone()
        bad[3, 5, 7] = float("nan")
        bad[9, :, :] = float("inf")
        got, _ = pl.plaid_search_vanilla(idx, bad, 2, 2000, 100)
        torch.cuda.synchronize()
        assert int(got.min()) >= -1 and int(got.max()) < 70_000
        clean = [q for q in range(16) if q not in (3, 9)]
        assert torch.equal(got[clean], ids[clean])
    finally:
        pl.plaid_index_free(idx)


@pytest.mark.parametrize("nbits", [1, 2])
def test_passages_around_the_chunks_of_a_list(nbits):
    """Lists that end within a group of eight, a step of 32 and a chunk of 64 tokens, and passages that fill a wave's list by themselves."""
    import paper_2205_09707_amd as pl
    import test_gpu_maxsim_lists as lists
    P = 52_000
    idx, a, g = lists._index(pl, P, 300, nbits, 11 + nbits)
    try:
        Q = torch.nn.functional.normalize(torch.randn(16, 32, 128, generator=g, device="cuda"), dim=2).contiguous()
        for nprobe, ncand in [(1, 7), (4, 13_000)]:
            got = pl.plaid_search_vanilla(idx, Q, nprobe, ncand, min(ncand, 500))
            want = pl.plaid_search_vanilla(idx, Q, nprobe, ncand, min(ncand, 500), debug=True)
            torch.cuda.synchronize()
            print("candidates", want[2]["n_cand"].tolist())
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    finally:
        pl.plaid_index_free(idx)
