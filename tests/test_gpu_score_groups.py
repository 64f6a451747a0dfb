"""Queries that a workgroup of the score kernel walks one after the other, in groups of one to eight with a shorter last one, get, bit for
bit, the scores and pruning bits that each gets in a launch of its own."""
import os
import shutil
import subprocess

import pytest
import torch

from test_build_properties import CSRC, HIPCC, ROOT

# queries and workgroups of one (256 centroids each): queries per workgroup
CLAIMS = ["scq16_queries(1, 1) == 1", "scq16_queries(1, 4096) == 1", "scq16_queries(512, 1) == 1", "scq16_queries(513, 1) == 2", "scq16_queries(23, 40) == 2",
          "scq16_queries(9, 128) == 3", "scq16_queries(16, 256) == 8", "scq16_queries(40, 128) == 5", "scq16_queries(6, 1024) == 6",
          "scq16_queries(256, 64) == 8", "scq16_queries(512, 256) == 64", "scq16_queries(512, 1024) == 64", "scq16_queries(144, 1024) == 64",
          "scq16_queries(100, 180) == 9",
          # all workgroups of one query at once, up to eight queries each
          "scq16_queries(5, 512) == 5", "scq16_queries(8, 512) == 8", "scq16_queries(9, 512) == 5", "scq16_queries(12, 256) == 6",
          "scq16_queries(32, 64) == 4", "scq16_queries(17, 256) == 5"]


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")), reason="hipcc not installed")
def test_queries_per_workgroup(tmp_path):
    unit = tmp_path / "rules.hip"
    unit.write_text('#include "k_scq16.hip"\n' + "".join(f'static_assert({c}, "{c}");\n' for c in CLAIMS))
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
                        "--cuda-host-only", "-fsyntax-only", str(unit)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("C,nq", [(300, 7), (10_007, 23), (33_000, 9), (33_000, 17), (70_000, 5), (70_000, 19)])
def test_scores_do_not_depend_on_the_group(C, nq):
    import paper_2205_09707_amd as pl
    g = torch.Generator(device="cuda")
    g.manual_seed(C + nq)
    P = 3000
    cen = torch.nn.functional.normalize(torch.randn(C, 128, generator=g, device="cuda"), dim=1).contiguous()
    offsets = torch.arange(P + 1, dtype=torch.int64, device="cuda") * 3
    codes = torch.randint(0, C, (3 * P,), generator=g, device="cuda", dtype=torch.int32)
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, offsets, C)
    arrays = {"centroids": cen, "doc_offsets": offsets, "codes": codes, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids,
              "residuals": torch.randint(0, 256, (3 * P, 32), generator=g, device="cuda", dtype=torch.uint8),
              "bucket_weights": torch.tensor([-0.05, -0.015, 0.015, 0.05], device="cuda")}
    idx = pl.plaid_index_from_view(arrays, 2, device=0, copy=False)
    try:
        Q = torch.nn.functional.normalize(cen[codes[:32 * nq].long()].reshape(nq, 32, 128) + 0.03 * torch.randn(nq, 32, 128, generator=g, device="cuda"), dim=2)
        want = ["S_cq", "keep", "probed"]
        _, _, all_ = pl.plaid_search_debug(idx, Q.contiguous(), 2, 0.4, 200, 10, want=want)
        for i in range(nq):
            _, _, one = pl.plaid_search_debug(idx, Q[i:i + 1].contiguous(), 2, 0.4, 200, 10, want=want)
            for name in want:
                assert torch.equal(one[name][0], all_[name][i]), (name, i)
    finally:
        pl.plaid_index_free(idx)
