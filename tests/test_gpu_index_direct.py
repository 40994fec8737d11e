"""The sort in one launch: positions around what a workgroup holds and what the launch takes, one and several workgroups to a unit,
windows, ids outside the range (dropped)."""
import numpy as np
import pytest
import torch

import paper_2502_08246_amd as saap
from oracle import ref
from synth import gen

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("units,N,B,slack,window", [
    (1, 4096, 64, 2, None), (3, 4097, 65, 1, None), (2, 8192, 16, 0, None), (2, 8193, 2048, 1, None), (1, 24577, 2047, 3, None),
    (2, 49152, 1000, 1, None), (1, 49153, 300, 1, None), (33, 16000, 40, 2, None), (64, 8200, 24, 1, None), (200, 9000, 16, 0, None),
    (2, 30000, 70, 2, (1, 2047)), (1, 10240, 33, 1, (1, 2047)), (1, 10241, 33, 0, (3, 1100)),
])
@pytest.mark.parametrize("dropped", [False, True])
def test_sort_in_one_launch(units, N, B, slack, window, dropped):
    rng = np.random.default_rng(N + B)
    ids = np.minimum(rng.geometric(8.0 / (B + 8), (1, units, N)) - 1, B - 1).astype(np.int32)
    K = torch.randn(1, units, N, 128, generator=torch.Generator(device=DEV).manual_seed(N), device=DEV).to(torch.bfloat16)
    build = (lambda i: saap.build_windowed_index(i, K, K, B, slack, *window)) if window else (lambda i: saap.build_bucket_index(i, K, K, B, slack))
    if dropped:                                            # what is left comes in the order that it has without the others
        out = ids.copy()
        at = rng.random(ids.shape) < 0.1
        if window:
            at[..., :window[0]], at[..., N - window[1]:] = False, False
        out[at] = rng.choice([-1, B, B + 7, 2 ** 31 - 1], int(at.sum()))
        off, ln, idx = (t.cpu().numpy()[0] for t in build(torch.from_numpy(out).to(DEV))[:3])
        for u in range(units):
            used = np.zeros(idx.shape[1], bool)
            for b in range(B):
                members = np.flatnonzero((out[0, u] == b) & (np.arange(N) >= window[0]) & (np.arange(N) < N - window[1]) if window else out[0, u] == b)
                assert ln[u, b] == len(members) and off[u, b + 1] - off[u, b] == len(members) + slack
                assert np.array_equal(idx[u, off[u, b]:off[u, b] + len(members)], members)
                used[off[u, b]:off[u, b] + len(members)] = True
            if window:
                used[off[u, B]:off[u, B] + sum(window)] = True
            assert (idx[u][~used] == -1).all()
        return
    got = build(torch.from_numpy(ids).to(DEV))
    hK = gen.to_host_f32(K)
    want = ref.build_windowed_index(ids, hK, hK, B, slack, *window) if window else ref.build_bucket_index(ids, hK, hK, B, slack)
    for g, w in zip(got[:3], want[:3]):
        assert np.array_equal(g.cpu().numpy(), w)
    if window:
        assert np.array_equal(got[5].cpu().numpy(), want[5])


@pytest.mark.parametrize("units,N,B,slack", [(3, 8193, 24, 1), (2, 20000, 70, 0), (1, 24577, 2048, 1), (2, 32768, 1, 2), (1, 32769, 9, 1)])
@pytest.mark.parametrize("kind", ["one id", "half one id", "two ids", "runs", "none in range", "last"])
def test_ids_that_many_positions_share(units, N, B, slack, kind):
    """Additions of a wave to one address: ids that most of its positions have, that change from run to run, or that no bucket has."""
    rng = np.random.default_rng(N + B)
    ids = rng.integers(0, B, (1, units, N)).astype(np.int32)
    if kind == "one id":
        ids[:] = B // 2
    if kind == "half one id":
        ids[rng.random(ids.shape) < 0.5] = B - 1
    if kind == "two ids":
        ids = np.where(rng.random(ids.shape) < 0.6, 0, B - 1).astype(np.int32)
    if kind == "runs":
        ids = np.broadcast_to((np.arange(N) // 300 * 7 % B).astype(np.int32), ids.shape).copy()
    if kind == "none in range":
        ids[rng.random(ids.shape) < 0.9] = -1
        ids[..., N // 2:] = B
    if kind == "last":
        ids[:], ids[..., N - 1] = 0, B - 1
    K = torch.zeros(1, units, N, 128, device=DEV, dtype=torch.bfloat16)
    off, ln, idx = (t.cpu().numpy()[0] for t in saap.build_bucket_index(torch.from_numpy(ids).to(DEV), K, K, B, slack)[:3])
    for u in range(units):
        kept = ids[0, u][(ids[0, u] >= 0) & (ids[0, u] < B)]
        assert np.array_equal(ln[u], np.bincount(kept, minlength=B)) and np.array_equal(np.diff(off[u]), ln[u] + slack) and off[u, 0] == 0
        want = np.full(idx.shape[1], -1, np.int32)
        at = np.argsort(np.where((ids[0, u] >= 0) & (ids[0, u] < B), ids[0, u], B), kind="stable")[:len(kept)]
        want[np.arange(len(kept)) + slack * np.sort(kept)] = at
        assert np.array_equal(idx[u], want)
