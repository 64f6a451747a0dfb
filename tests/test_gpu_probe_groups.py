"""The probes come from the maxima of 256-row groups (where there are more than 1024 tiles), of 32-row tiles and of rows in turn,
and rows that may be among the best are re-evaluated in double together: the probed centroids and the pruning map must be those
of the exact scores at the edges of the groups, past the 1024 groups that stay in registers, where rows repeat (more ties than a token's lists and than one
staging of rows hold) and for an index too small to lend the group maxima any memory."""
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [
    # C, copies of each row next to each other, passages
    (1, 1, 40), (31, 1, 40), (256, 1, 400), (257, 1, 400), (2049, 1, 400),
    (32_768, 1, 5000), (32_769, 1, 5000), (70_001, 1, 5000), (270_001, 1, 20_000),
    (513, 2, 400), (3000, 3, 400), (4096, 6, 400), (6000, 40, 400), (20_000, 300, 2000),
    (8000, 1, 20), (8000, 5, 20), (40_000, 1, 20),  # fewer than C / 16 passages
    (33_000, 3, 5000), (36_000, 40, 5000), (40_000, 300, 5000),  # ties with groups
]


@pytest.mark.parametrize("C,copies,P", CASES)
def test_probes_and_pruning_map_are_the_exact_ones(C, copies, P):
    import paper_2205_09707_amd as pl
    pl.load_library()
    g = torch.Generator(device="cuda")
    g.manual_seed(C + copies)
    cen = torch.nn.functional.normalize(torch.randn(-(-C // copies), 128, generator=g, device="cuda"), dim=1)
    cen = cen.repeat_interleave(copies, dim=0)[:C].contiguous()
    offsets = torch.arange(P + 1, dtype=torch.int64, device="cuda") * 5
    codes = torch.randint(0, C, (5 * P,), generator=g, device="cuda", dtype=torch.int32)
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, C)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.zeros(5 * P, 32, dtype=torch.uint8, device="cuda"),
              "bucket_weights": torch.linspace(-0.05, 0.05, 4, device="cuda")}
    Q = cen[torch.randint(0, C, (3 * 32,), generator=g, device="cuda")] + 0.03 * torch.randn(96, 128, generator=g, device="cuda")
    Q = torch.nn.functional.normalize(Q, dim=1).reshape(3, 32, 128).contiguous()
    idx = pl.plaid_index_from_view(arrays, 2, device=0, copy=False)
    try:
        for nprobe in (1, 2, 3, 4, 8):
            if nprobe > C:
                continue
            for t_cs in (0.5, 0.3):
                _, _, dbg = pl.plaid_search_debug(idx, Q, nprobe, t_cs, 50, 10, want=["probed", "keep"])
                for q in range(3):
                    S = (cen.double() @ Q[q].double().T).float()  # the definition's values: summed in double, rounded once
                    order = torch.sort(S, dim=0, descending=True, stable=True).indices  # ties to the smaller id
                    assert torch.equal(dbg["probed"][q], order[:nprobe].T.int()), (nprobe, t_cs, q)
                    bits = (dbg["keep"][q].unsqueeze(1) >> torch.arange(32, device="cuda", dtype=torch.int32)) & 1
                    assert torch.equal(bits.reshape(-1)[:C].bool(), S.max(dim=1).values >= t_cs), (nprobe, t_cs, q)
    finally:
        pl.plaid_index_free(idx)
