"""Where a single query's key list is in parts, and that the parts' places neither overlap nor leave the list; which lists are cut and scored
by one launch; which vectors are written past the caches.  On the GPU, a query whose list is in parts against the same one in a launch of
four, where none is."""
import os
import shutil
import subprocess

import pytest
import torch

from test_build_properties import CSRC, HIPCC, ROOT

PARTS = """
constexpr bool parts_fit(int64_t passages, int64_t P) {  // a workgroup's passages; at most S2_COPIES parts, each with its workgroups' places
    const int64_t blocks = (P + passages - 1) / passages;
    int64_t from[S2_COPIES] = {}, need[S2_COPIES] = {};
    for (int p = 0; p < S2_COPIES && p < blocks; ++p) {
        from[p] = s2_list_part(p, passages, P);
        for (int64_t b = p; b < blocks; b += S2_COPIES) need[p] += b + 1 < blocks ? passages : P - b * passages;
    }
    for (int p = 0; p < S2_COPIES && p < blocks; ++p) {
        if (from[p] < 0 || from[p] + need[p] > P) return false;
        for (int o = 0; o < p; ++o)
            if (from[p] < from[o] + need[o] && from[o] < from[p] + need[p]) return false;
    }
    return true;
}
"""


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not installed")
def test_rules_of_parts_and_cuts(tmp_path):
    claims = ["s2_parts(1, 481)", "!s2_parts(1, 480)", "!s2_parts(2, 4297)"]
    claims += [f"parts_fit({n}, {P})" for n in (128, 256, 512, 1024, 2048, 4096, 8192, 16384)
               for P in (1, 1023, 400_385, 405_003, 409_600, 800_769, 8 * 16384, 8 * 16384 + 1, 2_000_001, 8_800_000, (1 << 31) - 1)
               if P < 1_000_000 or n > 4096]
    for src, body in (("k_stage2.hip", PARTS + "".join(f'static_assert({c}, "{c}");\n' for c in claims)),
                      ("k_stage4.hip", "".join(f'static_assert({c}, "{c}");\n' for c in (
                          "s4_cuts(1024, 8)", "!s4_cuts(1024, 9)", "!s4_cuts(1025, 1)", "s4_cuts(256, 32)", "!s4_cuts(256, 33)", "s4_cuts(1, 8192)",
                          # what is written past the caches: more than the last of them holds, 256 MB
                          "!s4_past_caches(419430, true, true)", "s4_past_caches(419431, true, true)", "!s4_past_caches(524288, true, false)",
                          "s4_past_caches(524289, true, false)", "!s4_past_caches(2097152, false, true)", "s4_past_caches(2097153, false, true)",
                          "s4_past_caches(1ll << 40, true, true)", "!s4_past_caches(0, true, true)")))):
        unit = tmp_path / ("rules_" + src)
        unit.write_text(f'#include "{src}"\n' + body)
        r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-fconstexpr-steps=100000000", "-I" + os.path.join(ROOT, "include"),
                            "-I" + CSRC, "--cuda-host-only", "-fsyntax-only", str(unit)],
                           stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert r.returncode == 0, r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("P", [300_007, 409_600, 983_040, 983_041, 1_000_003])
def test_a_list_in_parts(P):
    """Around the smallest collection whose list is in parts, 481 ranges of 2048 passages; 300 007, with the largest ndocs below, in ranges of 512."""
    import paper_2205_09707_amd as pl
    C = 3000
    g = torch.Generator(device="cuda")
    g.manual_seed(P)
    cen = torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1)
    offsets = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cumsum(torch.randint(0, 5, (P,), generator=g, device="cuda"), 0)
    N = int(offsets[-1])
    codes = (torch.rand(N, generator=g, device="cuda") ** 3 * C).int().clamp_(max=C - 1)
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, C)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.randint(0, 256, (N, 16), generator=g, device="cuda", dtype=torch.uint8),
              "bucket_weights": torch.tensor([-0.05, 0.06], device="cuda")}
    Q = torch.nn.functional.normalize(cen[codes[torch.randint(0, N, (4 * 32,), generator=g, device="cuda")].long()]
                                      + 0.05 * torch.randn(4 * 32, 128, generator=g, device="cuda"), dim=1).reshape(4, 32, 128).contiguous()
    idx = pl.plaid_index_from_view(arrays, 1, device=0, copy=False)
    try:
        for nprobe, t_cs, ndocs in [(1, 0.5, 256), (4, 0.4, 4096), (2, 0.3, 60_000), (2, 0.99, 1024)]:
            pl.plaid_set_max_chunk(idx, 4)
            many = pl.plaid_search_debug(idx, Q, nprobe, t_cs, ndocs, 50, want=["n_cand", "n2", "sel3_ids", "n3"])
            pl.plaid_set_max_chunk(idx, 1)
            one = pl.plaid_search_debug(idx, Q, nprobe, t_cs, ndocs, 50, want=["n_cand", "n2", "sel3_ids", "n3"])
            ids, scores = pl.plaid_search(idx, Q, nprobe, t_cs, ndocs, 50)
            torch.cuda.synchronize()
            print(P, nprobe, "candidates", many[2]["n_cand"].tolist())
            for name in ("n_cand", "n2", "n3", "sel3_ids"):
                a, b = many[2][name], one[2][name]
                if name == "sel3_ids":  # (a set)
                    a, b = torch.sort(a, dim=1).values, torch.sort(b, dim=1).values
                assert torch.equal(a, b), (name, nprobe)
            for a, b in ((ids, scores), one[:2]):
                assert torch.equal(a, many[0]) and torch.equal(b, many[1]), nprobe
    finally:
        pl.plaid_index_free(idx)


@pytest.mark.gpu
@pytest.mark.parametrize("K,ndocs", [(32, 500), (58, 500), (32, 60_000), (58, 60_000)])
def test_a_list_in_parts_by_waves_with_more_areas(K, ndocs):
    """More surviving centroids without a bitmap than one wave's planes (26) or two waves' (52): a workgroup's passages are a half or a quarter
    then, and its part of the list is as much smaller."""
    import paper_2205_09707_amd as pl
    P, C = 1_000_003, 60_000
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    cen = torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1)
    offsets = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cumsum(torch.randint(0, 5, (P,), generator=g, device="cuda"), 0)
    N = int(offsets[-1])
    hot = 200  # centroids, 3000 passages each: in most ranges, and no list long enough for a bitmap
    codes = torch.randint(0, C, (N,), generator=g, device="cuda").int()
    some = torch.rand(N, generator=g, device="cuda") < 0.3
    codes[some] = torch.randint(0, hot, (int(some.sum()),), generator=g, device="cuda").int()
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, C)
    assert int((ivf_offsets[1:] - ivf_offsets[:-1]).max()) < P // 16
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.randint(0, 256, (N, 16), generator=g, device="cuda", dtype=torch.uint8),
              "bucket_weights": torch.tensor([-0.05, 0.06], device="cuda")}
    at = torch.stack([torch.randperm(hot, generator=g, device="cuda")[:K] for _ in range(4)])
    tok = torch.arange(32, device="cuda")  # a token at one centroid, or between two
    Q = cen[at[:, tok % K]] + (cen[at[:, 32 + tok % (K - 32)]] if K > 32 else 0)
    Q = torch.nn.functional.normalize(Q, dim=2).contiguous()
    idx = pl.plaid_index_from_view(arrays, 1, device=0, copy=False)
    try:
        pl.plaid_set_max_chunk(idx, 4)
        many = pl.plaid_search_debug(idx, Q, 2, 0.55, ndocs, 50, want=["n_cand", "n2", "n3", "sel2_ids", "keep"])
        assert sum((many[2]["keep"] >> s & 1).sum(1) for s in range(32)).tolist() == [K] * 4
        pl.plaid_set_max_chunk(idx, 1)
        one = pl.plaid_search_debug(idx, Q, 2, 0.55, ndocs, 50, want=["n_cand", "n2", "n3", "sel2_ids"])
        ids, scores = pl.plaid_search(idx, Q, 2, 0.55, ndocs, 50)
        torch.cuda.synchronize()
        assert int(many[2]["n_cand"].min()) > 4 * 480  # keys from many waves
        for name in ("n_cand", "n2", "n3"):
            assert torch.equal(many[2][name], one[2][name]), name
        for q in range(4):
            n = int(many[2]["n2"][q])  # (the kept ones are a set)
            assert torch.equal(torch.sort(many[2]["sel2_ids"][q, :n]).values, torch.sort(one[2]["sel2_ids"][q, :n]).values), q
        for a, b in ((ids, scores), one[:2]):
            assert torch.equal(a, many[0]) and torch.equal(b, many[1])
    finally:
        pl.plaid_index_free(idx)
