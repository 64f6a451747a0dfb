"""plaid_assign_centroids screens with one product of fp16 roundings and decides what that leaves open in double: the codes
must be the oracle's at the edges of its tiles (128 rows per wave, 512 per workgroup, 32 vectors per group), where many
centroids are nearly equal, and for values the fp16 roundings cannot hold (tiny, huge)."""
import numpy as np
import pytest
import torch

import test_gpu_index_build as tb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,n", [(1, 1), (127, 31), (128, 32), (129, 33), (512, 64), (513, 65), (1500, 700)])
@pytest.mark.parametrize("kind", ["unit", "clustered", "tiny", "long"])
def test_codes_equal_the_oracle(C, n, kind):
    import paper_2205_09707_amd as pl
    pl.load_library()
    rng = np.random.default_rng(1000 * C + n)
    cen = rng.standard_normal((C, 128))
    cen /= np.linalg.norm(cen, axis=1, keepdims=True)
    x = rng.standard_normal((n, 128))
    x /= np.linalg.norm(x, axis=1, keepdims=True)
    if kind == "clustered":    # centroids a few fp16 roundings apart: nearly every vector is decided in double
        cen = cen[:1] + 1e-4 * cen
    elif kind == "tiny":       # below fp16's normal range on both sides
        cen, x = cen * 1e-4, x * 1e-6
    elif kind == "long":       # norms up to 2^17: components past fp16's largest value among them
        x *= 2.0 ** rng.integers(-3, 18, size=(n, 1))
    cen, x = cen.astype(np.float32), x.astype(np.float32)
    want = tb._oracle_nearest(cen, x)
    got = pl.plaid_assign_centroids(torch.from_numpy(cen).cuda(), torch.from_numpy(x).cuda())
    torch.cuda.synchronize()
    np.testing.assert_array_equal(got.cpu().numpy(), want)
