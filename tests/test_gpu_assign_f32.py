"""fp32 key assignment on the matrix cores, keys of every kind beside each other in a workgroup of 128: keys whose best two centroids are equal
or nearly so, and keys whose scores are infinite or beyond fp32, as the last key of all (the lanes behind it hold copies of it) and elsewhere."""
import numpy as np
import pytest
import torch

import paper_2502_08246_amd as saap
from oracle import ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("N", [4097, 4200, 4223])         # 1, 104 and 127 keys in the last workgroup
@pytest.mark.parametrize("B", [16, 200])
@pytest.mark.parametrize("special", [float("inf"), float("-inf"), 3e38])
def test_close_keys_beside_infinite_scores(N, B, special):
    g = torch.Generator().manual_seed(N + B)
    c = torch.randn(2, B, 128, generator=g)
    c[:, 5] = c[:, 0]                                      # equal and nearly equal best centroids
    c[:, 9] = c[:, 0] * (1 + 2.0 ** -22)
    x = torch.randn(1, 2, N, 128, generator=g)
    x[:, :, ::3] = 0.1 * x[:, :, ::3] + c[:, :1]
    for at in (N - 1, N - 3, 4000, 130):
        x[0, :, at] = special * c[:, 0].sign() if abs(special) < 1e39 else x[0, :, at]
        if abs(special) > 1e39:
            x[0, :, at, 7] = special
    want = ref.assign_keys(x.numpy(), c.numpy(), None)
    assert np.array_equal(saap.assign_keys(x.to(DEV), c.to(DEV)).cpu().numpy(), want)
