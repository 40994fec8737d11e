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


@pytest.mark.parametrize("B", [2, 33, 255, 256, 257, 600])
@pytest.mark.parametrize("kind", ["few", "equal centroids", "zero centroids", "bias +inf", "tiny keys"])
def test_keys_scored_against_every_centroid(B, kind):
    """Four keys at a time: none to five of them in a workgroup, or all its keys."""
    g = torch.Generator().manual_seed(B)
    N = 4100
    c, x = torch.randn(2, B, 128, generator=g), torch.randn(1, 2, N, 128, generator=g)
    bias = None
    if kind == "few":
        for wg in range(N // 128):
            x[:, :, 128 * wg:128 * wg + wg % 6] *= 1e-18   # sums of squares too small to bound anything
        x[:, :, N - 3:] *= 1e-18
    if kind == "equal centroids":                          # more candidates than a workgroup lists
        c[:] = c[:, :1]
    if kind == "zero centroids":
        c = 0 * c
    if kind == "bias +inf":
        bias = torch.randn(2, B, generator=g)
        bias[:, B // 2] = bias[:, B - 1] = np.inf
    if kind == "tiny keys":
        x = x * 1e-18
    want = ref.assign_keys(x.numpy(), c.numpy(), None if bias is None else bias.numpy())
    assert np.array_equal(saap.assign_keys(x.to(DEV), c.to(DEV), None if bias is None else bias.to(DEV)).cpu().numpy(), want)


@pytest.mark.parametrize("close", [1, 2, 3, 8, 9, 127])
def test_few_close_keys_and_many(close):
    """Up to eight close keys of a workgroup are scored against every centroid, one or two of them another way than more, and more than eight against the
    centroids they list."""
    g = torch.Generator().manual_seed(close)
    c = torch.randn(1, 300, 128, generator=g)
    c[:, 7] = c[:, 250] * (1 + 2.0 ** -22)
    c[:, 77] = c[:, 250]
    x = 0.05 * torch.randn(1, 1, 4000, 128, generator=g) + 3 * c[:, torch.arange(4000) % 70 + 8][None]
    for wg in range(32):
        at = torch.arange(128 * wg, min(128 * wg + close, 4000))
        x[:, :, at] = 3 * c[:, 250] + 1e-4 * torch.randn(1, 1, len(at), 128, generator=g)
    want = ref.assign_keys(x.numpy(), c.numpy(), None)
    assert np.array_equal(saap.assign_keys(x.to(DEV), c.to(DEV)).cpu().numpy(), want)


@pytest.mark.parametrize("S,Hkv,N", [(512, 8, 1), (512, 8, 4), (512, 8, 5), (700, 1, 5), (700, 1, 6), (2, 1, 1024), (3, 1, 683), (1, 3, 1)])
@pytest.mark.parametrize("B", [3, 40])
def test_few_keys_of_many_heads(S, Hkv, N, B):
    """Numbers of keys on both sides of the line between a workgroup per key and a workgroup per 128 keys of a head, on a device of 256
    compute units."""
    g = torch.Generator().manual_seed(S * N + B)
    c, x = torch.randn(Hkv, B, 128, generator=g), torch.randn(S, Hkv, N, 128, generator=g)
    c[:, B - 1] = c[:, 0]
    want = ref.assign_keys(x.numpy(), c.numpy(), None)
    assert np.array_equal(saap.assign_keys(x.to(DEV), c.to(DEV)).cpu().numpy(), want)
