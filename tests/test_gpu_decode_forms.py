"""plaid_decompress_passages on collections of short and of longer passages: passages of lengths around the rows that a workgroup's threads have in
flight, lists around the ids of one of the offsets kernel's workgroups (64) and around a workgroup per compute unit (16 384), with and without
bucket indices and unit lengths."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbits", [1, 2])
@pytest.mark.parametrize("lengths", [[0, 1, 7, 8, 9, 31, 32, 33, 65], [0, 1, 15, 16, 17, 63, 64, 65, 130], [24], [23]])
def test_lists_and_lengths(nbits, lengths):
    import paper_2205_09707_amd as pl
    P, C = 1000, 64
    g = torch.Generator(device="cuda")
    g.manual_seed(P + nbits)
    n_tok = torch.tensor(lengths, device="cuda")[torch.arange(P, device="cuda") % len(lengths)]
    offsets = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cumsum(n_tok, 0)
    N = int(offsets[-1])
    assert (N >= 24 * P) == (lengths in ([0, 1, 15, 16, 17, 63, 64, 65, 130], [24]))
    codes = torch.randint(0, C, (N,), generator=g, device="cuda", dtype=torch.int32)
    io, ip = pl.plaid_build_ivf(codes, offsets, C)
    cen = torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1).contiguous()
    res = torch.randint(0, 256, (N, 16 * nbits), generator=g, device="cuda", dtype=torch.uint8)
    w = torch.linspace(-0.06, 0.05, 1 << nbits, device="cuda")
    idx = pl.plaid_index_from_view({"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": io, "ivf_pids": ip, "residuals": res,
                                    "bucket_weights": w}, nbits, device=0, copy=False)
    try:
        shifts = range(8 - nbits, -1, -nbits)
        all_ind = torch.stack([(res >> s) & ((1 << nbits) - 1) for s in shifts], dim=2).reshape(N, 128)
        all_vec = cen[codes.long()] + w[all_ind.long()]
        for n in (1, 64, 65, 129, 16_384, 16_385):
            pids = (torch.arange(n, device="cuda") * 7 + 5) % P
            length = offsets[pids + 1] - offsets[pids]
            want = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
            want[1:] = torch.cumsum(length, 0)
            total = int(want[-1])
            tok = torch.repeat_interleave(offsets[pids] - want[:-1], length) + torch.arange(total, device="cuda")
            for indices in (True, False):
                offs, vec, ind = pl.plaid_decompress_passages(idx, pids.int(), total, indices=indices)
                torch.cuda.synchronize()
                assert torch.equal(offs, want) and torch.equal(vec, all_vec[tok]), n
                assert not indices or torch.equal(ind, all_ind[tok]), n
        pl.plaid_index_set_renormalize(idx, True)
        vec = pl.plaid_decompress_passages(idx, pids.int(), total)[1]
        # a factor of one rounding of a square root's reciprocal, and one rounding per component
        assert float((vec - torch.nn.functional.normalize(all_vec.double(), dim=1)[tok]).abs().max()) < 3 * 2.0 ** -24
    finally:
        pl.plaid_index_free(idx)


def test_short_passages_of_a_long_collection_take_no_longer():
    """What a list costs depends on its passages, not on the others of the collection: the same 50 000 of 8 to 24 tokens, alone and beside as many of
    60 to 100.  (With workgroups by the collection's mean the second took 1.5 times as long.)"""
    import paper_2205_09707_amd as pl
    C, half = 4096, 100_000
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    short = torch.randint(8, 25, (half,), generator=g, device="cuda")
    cen = torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1).contiguous()
    pids = torch.randint(0, half, (50_000,), generator=g, device="cuda").int()
    total = int(short[pids.long()].sum())
    indices = []
    for lengths in (short, torch.cat([short, torch.randint(60, 101, (half,), generator=g, device="cuda")])):
        offsets = torch.zeros(lengths.numel() + 1, dtype=torch.int64, device="cuda")
        offsets[1:] = torch.cumsum(lengths, 0)
        N = int(offsets[-1])
        codes = torch.randint(0, C, (N,), generator=g, device="cuda", dtype=torch.int32)
        io, ip = pl.plaid_build_ivf(codes, offsets, C)
        indices.append(pl.plaid_index_from_view({"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": io, "ivf_pids": ip,
                                                 "residuals": torch.randint(0, 256, (N, 32), generator=g, device="cuda", dtype=torch.uint8),
                                                 "bucket_weights": torch.linspace(-0.06, 0.05, 4, device="cuda")}, 2, device=0, copy=False))
    try:
        times = [[], []]
        for _ in range(15):
            for idx, t in zip(indices, times):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                pl.plaid_decompress_passages(idx, pids, total)
                a.record()
                for _ in range(8):
                    pl.plaid_decompress_passages(idx, pids, total)
                b.record()
                torch.cuda.synchronize()
                t.append(a.elapsed_time(b))
        alone, beside = (sorted(t)[7] for t in times)
        print(f"50 000 short passages: {1000 * alone / 8:.0f} us a call, of a longer collection {1000 * beside / 8:.0f}")
        assert beside < 1.2 * alone
    finally:
        for idx in indices:
            pl.plaid_index_free(idx)


@pytest.mark.parametrize("nbits", [1, 2])
@pytest.mark.parametrize("vectors,indices,tokens", [(True, True, 419_430), (True, True, 419_431), (True, False, 524_288), (True, False, 524_289),
                                                    (False, True, 2_097_152), (False, True, 2_097_153)])
def test_outputs_through_the_caches_and_past_them(nbits, vectors, indices, tokens):
    """256 MB and a token more: what the list's passages hold decides, not the caller's capacity, which is twice that here."""
    import paper_2205_09707_amd as pl
    C = 512
    g = torch.Generator(device="cuda")
    g.manual_seed(tokens)
    lengths = torch.cat([torch.full((2000,), 64, device="cuda"), torch.ones(64, dtype=torch.int64, device="cuda")])
    offsets = torch.zeros(lengths.numel() + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cumsum(lengths, 0)
    N = int(offsets[-1])
    codes = torch.randint(0, C, (N,), generator=g, device="cuda", dtype=torch.int32)
    io, ip = pl.plaid_build_ivf(codes, offsets, C)
    cen = torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1).contiguous()
    res = torch.randint(0, 256, (N, 16 * nbits), generator=g, device="cuda", dtype=torch.uint8)
    w = torch.linspace(-0.06, 0.05, 1 << nbits, device="cuda")
    idx = pl.plaid_index_from_view({"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": io, "ivf_pids": ip, "residuals": res,
                                    "bucket_weights": w}, nbits, device=0, copy=False)
    try:
        pids = torch.cat([torch.arange(tokens // 64, device="cuda") * 7 % 2000, 2000 + torch.arange(tokens % 64, device="cuda")])
        length = offsets[pids + 1] - offsets[pids]
        want = torch.zeros(pids.numel() + 1, dtype=torch.int64, device="cuda")
        want[1:] = torch.cumsum(length, 0)
        assert int(want[-1]) == tokens
        tok = torch.repeat_interleave(offsets[pids] - want[:-1], length) + torch.arange(tokens, device="cuda")
        offs, vec, ind = pl.plaid_decompress_passages(idx, pids.int(), 2 * tokens, vectors=vectors, indices=indices)
        torch.cuda.synchronize()
        assert torch.equal(offs, want)
        all_ind = torch.stack([(res >> s) & ((1 << nbits) - 1) for s in range(8 - nbits, -1, -nbits)], dim=2).reshape(N, 128)
        if vectors:
            assert torch.equal(vec[:tokens], (cen[codes.long()] + w[all_ind.long()])[tok])
        if indices:
            assert torch.equal(ind[:tokens], all_ind[tok])
    finally:
        pl.plaid_index_free(idx)
