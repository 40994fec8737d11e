"""The bucket of an appended key where fp32 scores do not decide it: equal and nearly equal centroids inside a slab of 128 and in
several, rows of zeros, values next to nothing, several rounds to a workgroup, and a key that starts on an odd element."""
import numpy as np
import pytest
import torch

import paper_2502_08246_amd as saap
from oracle import ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def centroids(kind, Hkv, B, dtype, g):
    c = torch.randn(Hkv, B, 128, generator=g)
    c /= c.norm(dim=-1, keepdim=True)
    c = c.to(dtype)
    win = min(B - 1, 77)
    close = c[:, win].clone()
    close[:, 5] = close[:, 5] * (1 + 2.0 ** -7)          # one unit in the last place of bfloat16, or a little in fp32
    places = {"random": [], "pair": [0, B - 1], "close": [3, B // 2], "many": range(0, B, 2), "zeros": [], "tiny": [1], "huge": [2]}[kind]
    for i, b in enumerate(b for b in places if b < B):
        if b != win:
            c[:, b] = close if kind == "close" and i == 0 else c[:, win]
    if kind == "zeros":
        c[:, ::3] = 0
    x = c[:, win].float() * 30
    if kind == "tiny":
        x, c = x * 2.0 ** -70, (c.float() * 2.0 ** -60).to(dtype)
    if kind == "huge":
        x, c = x * 2.0 ** 60, (c.float() * 2.0 ** 60).to(dtype)
    return x.to(dtype), c


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("S,Hkv,B", [(1, 2, 1), (2, 2, 100), (1, 1, 128), (1, 3, 129), (2, 2, 300), (1, 8, 1024), (64, 8, 600), (1, 2, 4100)])
@pytest.mark.parametrize("kind", ["random", "pair", "close", "many", "zeros", "tiny", "huge"])
@pytest.mark.parametrize("biased", [False, True])
def test_bucket_of_an_appended_key(dtype, S, Hkv, B, kind, biased):
    g = torch.Generator().manual_seed(B + S)
    x, c = centroids(kind, Hkv, B, dtype, g)
    keys = (x.float().unsqueeze(0) + (0.02 * x.float().abs().mean()) * torch.randn(S, Hkv, 128, generator=g) * (kind != "pair")).to(dtype)
    bias = 1e-3 * torch.randn(Hkv, B, generator=g) if biased else None
    want = ref.assign_keys(keys.float().unsqueeze(2).numpy(), c.float().numpy(), None if bias is None else bias.numpy())[:, :, 0]
    N, slack = 16, 1
    K = torch.zeros(S, Hkv, N, 128, dtype=dtype, device=DEV)
    off, ln, idx, Ks, Vs = saap.build_bucket_index(torch.zeros(S, Hkv, N, dtype=torch.int32, device=DEV), K, K, B, slack)
    room = torch.zeros(S * Hkv * 128 + 1, dtype=dtype, device=DEV)
    x_new = room[1:].view(S, Hkv, 128)
    x_new.copy_(keys)
    new = torch.randn(S, Hkv, 128, generator=g).to(dtype).to(DEV)
    pos = torch.full((S,), N, dtype=torch.int32, device=DEV)
    for _ in range(2):                                     # the counters of the workgroups are back at zero
        before = ln.clone()
        ids, flag = saap.append_keys(x_new, new, new, pos, c.to(DEV), None if bias is None else bias.to(DEV), off, ln, idx, Ks, Vs)
        assert np.array_equal(ids.cpu().numpy(), want)
        grown = (ln - before).cpu()
        assert flag[0].item() == 1 or torch.equal(grown.nonzero()[:, 2].view(S, Hkv), torch.from_numpy(want).long())
        ln.copy_(before)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("S,Hkv,B", [(1, 2, 100), (2, 2, 300), (64, 8, 600), (1, 2, 4100)])
@pytest.mark.parametrize("kind", ["some masked", "all masked", "one left", "+inf", "zero key", "zero key biased", "equal rows", "masked zeros", "lowest"])
def test_scores_that_are_known_or_equal(dtype, S, Hkv, B, kind):
    """Biases of infinity, keys of zeros, whole slabs of equal rows: no candidate, one and many in a slab, in one slab and in all."""
    g = torch.Generator().manual_seed(B)
    c, x = torch.randn(Hkv, B, 128, generator=g), 3 * torch.randn(S, Hkv, 128, generator=g)
    bias = torch.randn(Hkv, B, generator=g)
    if kind == "some masked":
        bias[:, ::2] = -np.inf
    if kind in ("all masked", "one left"):
        bias[:] = -np.inf
    if kind == "one left":
        bias[:, B - 3] = -5.0
    if kind == "+inf":
        bias[:, [B - 1, B // 2, 40]] = np.inf
    if kind.startswith("zero key"):
        x = 0 * x
    if kind == "zero key":
        bias = None
    if kind == "equal rows":
        c[:], bias = c[:, B // 2:B // 2 + 1].clone(), None
    if kind == "masked zeros":
        c[:, 7:], bias[:, ::3] = 0, -np.inf
    if kind == "lowest":
        bias[:] = torch.finfo(torch.float32).min
    x, c = x.to(dtype), c.to(dtype)
    want = ref.assign_keys(x.float().unsqueeze(2).numpy(), c.float().numpy(), None if bias is None else bias.numpy())[:, :, 0]
    K = torch.zeros(S, Hkv, 16, 128, dtype=dtype, device=DEV)
    off, ln, idx, Ks, Vs = saap.build_bucket_index(torch.zeros(S, Hkv, 16, dtype=torch.int32, device=DEV), K, K, B, 1)
    x, pos = x.to(DEV), torch.full((S,), 16, dtype=torch.int32, device=DEV)
    bias = None if bias is None else bias.to(DEV)
    for _ in range(2):
        before = ln.clone()
        ids, _ = saap.append_keys(x, x, x, pos, c.to(DEV), bias, off, ln, idx, Ks, Vs)
        assert np.array_equal(ids.cpu().numpy(), want)
        ln.copy_(before)
    off, ln, idx, Ks, Vs, rid = saap.build_windowed_index(torch.zeros(S, Hkv, 16, dtype=torch.int32, device=DEV), K, K, B, 1, 1, 7)
    ids, flag = saap.window_push(x, x, x, pos, c.to(DEV), bias, off, ln, idx, Ks, Vs, rid, 1, 7)
    assert np.array_equal(ids.cpu().numpy(), want)


def test_scores_that_are_no_numbers_have_one_outcome():
    """The definition leaves the bucket open; the same inputs have the same one, in the range, every time."""
    g = torch.Generator().manual_seed(0)
    c, x = torch.randn(8, 1024, 128, generator=g), torch.randn(8, 8, 128, generator=g)
    c[:, [5, 69, 300, 400, 401, 402]] = np.nan
    x, c, pos = x.to(DEV), c.to(DEV), torch.full((8,), 16, dtype=torch.int32, device=DEV)
    K = torch.zeros(8, 8, 16, 128, device=DEV)
    off, ln, idx, Ks, Vs = saap.build_bucket_index(torch.zeros(8, 8, 16, dtype=torch.int32, device=DEV), K, K, 1024, 1)
    before, seen = ln.clone(), []
    for _ in range(20):
        seen.append(saap.append_keys(x, x, x, pos, c, None, off, ln, idx, Ks, Vs)[0].clone())
        ln.copy_(before)
    assert all(torch.equal(s, seen[0]) for s in seen) and ((seen[0] >= 0) & (seen[0] < 1024)).all()
