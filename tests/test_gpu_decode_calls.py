"""plaid_decompress_passages: ids out of range at the edges of the offsets kernel's workgroups (1024 ids) and rounds (4096) are
refused with their place, leave the outputs alone and nothing on the stream, and the index serves the next call; lists around a
round's length; a stream with work before the call; several threads with streams of their own."""
import ctypes as ct
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu


def _index(pl, P, nbits=2):
    g = torch.Generator(device="cuda")
    g.manual_seed(P)
    C = 64
    lengths = torch.randint(0, 9, (P,), generator=g, device="cuda")
    offsets = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cumsum(lengths, 0)
    N = int(offsets[-1])
    codes = torch.randint(0, C, (N,), generator=g, device="cuda", dtype=torch.int32)
    io, ip = pl.plaid_build_ivf(codes, offsets, C)
    arrays = {"centroids": torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1).contiguous(),
              "doc_offsets": offsets, "codes": codes, "ivf_offsets": io, "ivf_pids": ip,
              "residuals": torch.randint(0, 256, (N, 16 * nbits), generator=g, device="cuda", dtype=torch.uint8),
              "bucket_weights": torch.tensor([-0.05, -0.015, 0.015, 0.05][:1 << nbits], device="cuda")}
    return pl.plaid_index_from_view(arrays, nbits, device=0, copy=False), arrays


def _expected(arrays, pids):
    o = arrays["doc_offsets"]
    tok = torch.cat([torch.arange(int(o[p]), int(o[p + 1]), device="cuda") for p in pids.tolist()] or [torch.empty(0, dtype=torch.int64, device="cuda")])
    r = arrays["residuals"][tok].int()
    ind = torch.stack([(r >> s) & 3 for s in (6, 4, 2, 0)], dim=2).reshape(len(tok), 128)
    return arrays["centroids"][arrays["codes"][tok].long()] + arrays["bucket_weights"][ind], ind.byte()


@pytest.mark.parametrize("n", [0, 1, 63, 1023, 1025, 4096, 4097, 16_385])
def test_lists_around_a_round(n):
    import paper_2205_09707_amd as pl
    idx, arrays = _index(pl, 3000)
    try:
        pids = (torch.arange(n, device="cuda") * 37 % 3000).int()
        o = arrays["doc_offsets"]
        want = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
        want[1:] = torch.cumsum(o[pids.long() + 1] - o[pids.long()], 0)
        total = int(want[-1])
        offs, vec, ind = pl.plaid_decompress_passages(idx, pids, total)
        assert torch.equal(offs, want)
        few = pids[:300]
        v, i = _expected(arrays, few)
        assert torch.equal(vec[:len(v)], v) and torch.equal(ind[:len(i)], i)
        if total:
            with pytest.raises(RuntimeError, match="capacity"):
                pl.plaid_decompress_passages(idx, pids, total - 1)
    finally:
        pl.plaid_index_free(idx)


@pytest.mark.parametrize("n,places", [(1, [0]), (100, [99]), (4096, [4095]), (4097, [4096]), (20_000, [1024, 19_999]), (20_000, [5, 8191, 16_384])])
@pytest.mark.parametrize("value", [-1, 3000, 2**31 - 1])
def test_ids_out_of_range_are_refused(n, places, value):
    import paper_2205_09707_amd as pl
    idx, arrays = _index(pl, 3000)
    try:
        pids = (torch.arange(n, device="cuda") * 7 % 3000).int()
        bad = pids.clone()
        bad[places] = value
        with pytest.raises(RuntimeError, match=rf"pids\[{places[0]}\] = {value} out of range"):
            pl.plaid_decompress_passages(idx, bad, 9 * n)
        assert int(pl.plaid_decompress_passages(idx, pids, 9 * n)[0][-1]) > 0  # the index serves the next call
    finally:
        pl.plaid_index_free(idx)


@pytest.mark.parametrize("n", [1, 1025, 20_000])
def test_a_refused_call_leaves_the_outputs_alone(n):
    """... and nothing on the stream, whose caller may use the buffers again from elsewhere."""
    import paper_2205_09707_amd as pl
    idx, arrays = _index(pl, 3000)
    lib = pl.load_library()
    try:
        pids = (torch.arange(n, device="cuda") * 7 % 3000).int()
        o = arrays["doc_offsets"]
        want = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
        want[1:] = torch.cumsum(o[pids.long() + 1] - o[pids.long()], 0)
        total = int(want[-1])
        assert total > 0
        bad = pids.clone()
        bad[n // 2] = 3000
        offs = torch.full((n + 1,), 77, dtype=torch.int64, device="cuda")
        vec = torch.full((total, 128), 7.0, device="cuda")
        ind = torch.full((total, 128), 9, dtype=torch.uint8, device="cuda")
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()

        def call(list_, capacity, vectors=True):
            p = [ct.c_void_p(t.data_ptr()) for t in (list_, offs, vec, ind)]
            return lib.plaid_decompress_passages(idx.handle, p[0], n, p[1], p[2] if vectors else None, p[3] if vectors else None,
                                                 capacity, ct.c_void_p(stream.cuda_stream))

        def untouched():
            return bool((vec == 7.0).all()) and bool((ind == 9).all())

        assert call(bad, total) == -1 and "out of range" in pl.plaid_last_error()
        assert stream.query() and untouched() and bool((offs == 77).all())
        assert call(bad, 0, vectors=False) == -1
        stream.synchronize()
        assert bool((offs == 77).all())
        assert call(pids, total - 1) == -1 and "capacity" in pl.plaid_last_error()
        assert stream.query() and untouched() and torch.equal(offs, want)
        offs.fill_(77)
        torch.cuda.synchronize()
        assert call(pids, 0, vectors=False) == 0  # (no rows asked for: the capacity does not matter)
        stream.synchronize()
        assert torch.equal(offs, want)
        assert call(pids, total) == 0
        stream.synchronize()
        v, i = _expected(arrays, pids[:300])
        assert torch.equal(vec[:len(v)], v) and torch.equal(ind[:len(i)], i)
    finally:
        pl.plaid_index_free(idx)


def test_a_busy_stream_is_not_waited_for_past_the_report():
    """Behind several milliseconds of other work the call returns with the report, before the vectors (5 GB of them) are there."""
    import paper_2205_09707_amd as pl
    idx, arrays = _index(pl, 3000)
    try:
        pids = (torch.arange(2_000_000, device="cuda") * 7 % 3000).int()
        o = arrays["doc_offsets"]
        total = int((o[pids.long() + 1] - o[pids.long()]).sum())
        pl.plaid_decompress_passages(idx, pids, total)
        torch.cuda.synchronize()
        torch.cuda._sleep(20_000_000)
        offs, vec, ind = pl.plaid_decompress_passages(idx, pids, total)
        assert not torch.cuda.current_stream().query()
        v, i = _expected(arrays, pids[:300])
        assert int(offs[-1]) == total and torch.equal(vec[:len(v)], v) and torch.equal(ind[:len(i)], i)
    finally:
        pl.plaid_index_free(idx)


def test_refused_under_capture():
    import paper_2205_09707_amd as pl
    idx, arrays = _index(pl, 3000)
    pids = torch.arange(10, device="cuda", dtype=torch.int32)
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    try:
        with torch.cuda.graph(graph, stream=stream):
            x = torch.ones(4, device="cuda")
            with pytest.raises(RuntimeError):
                pl.plaid_decompress_passages(idx, pids, 90)
            y = x + 1
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, torch.full((4,), 2.0, device="cuda"))
    finally:
        pl.plaid_index_free(idx)


def test_several_threads():
    """Lists of their own, one thread with an id out of range and one with too little room now and then: each call reports on its
    own list."""
    import paper_2205_09707_amd as pl
    idx, arrays = _index(pl, 3000)
    wrong, done = [], []

    def work(t):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                pids = (torch.arange(50 + 700 * t, device="cuda") * (11 + t) % 3000).int()
                bad = pids.clone()
                bad[t] = -5 - t
                v, i = _expected(arrays, pids)
                torch.cuda.current_stream().synchronize()
                for r in range(20):
                    offs, vec, ind = pl.plaid_decompress_passages(idx, pids, len(v))
                    if not (int(offs[-1]) == len(v) and torch.equal(vec, v) and torch.equal(ind, i)):
                        wrong.append((t, r))
                    if t == 1:
                        with pytest.raises(RuntimeError, match=rf"pids\[{t}\] = {-5 - t} out of range"):
                            pl.plaid_decompress_passages(idx, bad, len(v))
                    if t == 2:
                        with pytest.raises(RuntimeError, match=f"passages hold {len(v)} tokens, capacity is {len(v) - 1}"):
                            pl.plaid_decompress_passages(idx, pids, len(v) - 1)
                    done.append(t)
                torch.cuda.current_stream().synchronize()
        except BaseException as e:
            wrong.append((t, repr(e)))

    try:
        torch.cuda.synchronize()
        threads = [threading.Thread(target=work, args=(t,)) for t in range(5)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not wrong and len(done) == 100
    finally:
        pl.plaid_index_free(idx)
