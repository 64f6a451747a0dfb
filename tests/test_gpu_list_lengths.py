"""plaid_build_ivf sorts a list in the registers of a wave (up to 2048 passages; 1 to 32 a lane) or in a bitmap: lists of the lengths around a
lane's numbers of entries, passages in no order, centroids that occur more than once in a passage."""
import pytest
import torch

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 2, 3, 4, 5, 8, 9, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025,
           1500, 2047, 2048, 2049, 3000]


@pytest.mark.parametrize("P", [3000, 70_001])
def test_lists_of_every_form(P):
    import paper_2205_09707_amd as pl
    pl.load_library()
    g = torch.Generator(device="cuda")
    g.manual_seed(P)
    lists = [torch.sort(torch.randperm(P, generator=g, device="cuda")[:n]).values for n in LENGTHS]
    pids = torch.cat(lists + [lists[9], lists[20]])  # two of them twice
    cents = torch.cat([torch.full((len(l),), c, device="cuda") for c, l in enumerate(lists + [lists[9], lists[20]])])
    cents[cents == len(lists)] = 9
    cents[cents == len(lists) + 1] = 20
    order = torch.sort(pids, stable=True).indices
    codes = cents[order].int()
    offsets = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cumsum(torch.bincount(pids, minlength=P), 0)
    for _ in range(3):
        ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, len(LENGTHS) + 1)
        torch.cuda.synchronize()
        assert ivf_offsets.tolist() == [sum(LENGTHS[:c]) for c in range(len(LENGTHS) + 1)] + [sum(LENGTHS)]
        assert torch.equal(ivf_pids[:sum(LENGTHS)].long(), torch.cat(lists))
