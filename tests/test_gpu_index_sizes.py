"""Index builds at the sizes where the sort changes its shape (one launch for short contexts, slices beyond) and at the
edges of its rounds and slices, zeroed free slots included, against the oracle; keys whose ids lie outside the range,
with what the outputs held before the call at its worst; the centroid step from bucket ids against the one from grouped
features, bit for bit."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import ref
from synth import gen

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def saap():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the -m gpu tests need a real device")
    import paper_2502_08246_amd as lib
    lib.load_library()
    return lib


@pytest.mark.parametrize("N,B,slack,window", [
    (1, 16, 0, None), (63, 16, 3, None), (1025, 17, 2, None), (16384, 2048, 1, None), (16383, 2047, 65, None),
    (16385, 48, 2, None), (16384, 2049, 1, None), (20481, 4096, 0, None), (30000, 1, 5, None),
    (100, 16, 2, (4, 200)), (5000, 33, 2, (1, 2047)), (18433, 33, 1, (1, 2047)), (2048, 16, 0, (1, 2047)), (3000, 16, 4, (0, 0))])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_index_of_odd_sizes(saap, N, B, slack, window, dtype):
    if dtype == "f32" and N > 17000:
        pytest.skip("row copies of either width share the order of the keys")
    rng = np.random.default_rng(N + B)
    S, Hkv = 1, 2
    # most keys in a few buckets, some buckets empty
    ids = np.minimum(rng.geometric(8.0 / (B + 8), (S, Hkv, N)) - 1, B - 1).astype(np.int32)
    K = torch.randn(S, Hkv, N, 128, generator=torch.Generator(device=DEV).manual_seed(N), device=DEV).to(gen.torch_dtype(dtype))
    V = -K
    d_ids = torch.from_numpy(ids).to(DEV)
    hK, hV = gen.to_host_f32(K), gen.to_host_f32(V)
    junk = torch.full((4 * K.numel(),), 7.0, device=DEV)          # the caching allocator hands this memory out again
    del junk
    if window:
        got = saap.build_windowed_index(d_ids, K, V, B, slack, *window)
        want = ref.build_windowed_index(ids, hK, hV, B, slack, *window)
        assert np.array_equal(got[5].cpu().numpy(), want[5])
    else:
        got = saap.build_bucket_index(d_ids, K, V, B, slack)
        want = ref.build_bucket_index(ids, hK, hV, B, slack)
    for g, w in zip(got[:3], want[:3]):
        assert np.array_equal(g.cpu().numpy(), w)
    live = want[2] >= 0
    for g, w in zip(got[3:5], want[3:5]):
        g = gen.to_host_f32(g)
        assert np.array_equal(g[live], w[live]) and not g[~live].any()


@pytest.mark.parametrize("N,B,slack,window", [
    (700, 16, 0, None), (5000, 33, 3, None), (20481, 48, 0, None), (30000, 4096, 2, None),
    (900, 16, 0, (1, 100)), (5003, 33, 2, (4, 300)), (30000, 64, 1, (1, 2047)), (300, 16, 2, (1, 500))])
@pytest.mark.parametrize("zeroed", [True, False])
def test_ids_outside_the_range_are_dropped(saap, N, B, slack, window, zeroed):
    """Every slot that no key takes is marked, the slots the dropped keys leave behind the last run among them, whatever
    idx held before; free rows are zero or, from the call that does not zero, as they were."""
    rng = np.random.default_rng(N)
    S, Hkv = 2, 2
    ids = rng.integers(0, B, (S, Hkv, N)).astype(np.int32)
    wrong = rng.random((S, Hkv, N)) < np.array([0.0, 0.01, 0.3, 1.0]).reshape(S, Hkv, 1)      # of a unit: none to all
    ids[wrong] = rng.choice(np.array([-1, B, -2 ** 31, 2 ** 30], np.int32), int(wrong.sum()))
    K = torch.randn(S, Hkv, N, 128, generator=torch.Generator(device=DEV).manual_seed(N), device=DEV).to(torch.bfloat16)
    V = -K
    hK, hV = gen.to_host_f32(K), gen.to_host_f32(V)
    want = ref.build_windowed_index(ids, hK, hV, B, slack, *window) if window else ref.build_bucket_index(ids, hK, hV, B, slack)
    Ncap = want[2].shape[2]
    off, ln = (torch.empty(w.shape, dtype=torch.int32, device=DEV) for w in want[:2])
    idx = torch.full((S, Hkv, Ncap), 2 ** 30, dtype=torch.int32, device=DEV)
    Ks, Vs = (torch.full((S, Hkv, Ncap, 128), 7.0, dtype=torch.bfloat16, device=DEV) for _ in range(2))
    d_ids = torch.from_numpy(ids).to(DEV)
    ws = torch.zeros(saap.workspace_bytes(1, S=S, Hkv=Hkv, N=N, B=B), dtype=torch.uint8, device=DEV)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    ints = lambda *v: [ctypes.c_int32(i) for i in v]  # noqa: E731
    head = [ptr(t) for t in (d_ids, K, V, off, ln, idx, Ks, Vs)]
    tail = [ptr(ws), ctypes.c_size_t(ws.numel()), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)]
    suffix = "_zeroed" if zeroed else ""
    if window:
        res = torch.empty(want[5].shape, dtype=torch.int32, device=DEV)
        st = getattr(saap.load_library(), "saap_build_windowed_index" + suffix)(
            *head, ptr(res), *ints(S, Hkv, N, Ncap, B, 128, saap.BF16, slack, *window), *tail)
        assert np.array_equal(res.cpu().numpy(), want[5])
    else:
        st = getattr(saap.load_library(), "saap_build_bucket_index" + suffix)(
            *head, *ints(S, Hkv, N, Ncap, B, 128, saap.BF16, slack), *tail)
    assert st == 0
    for g, w in zip((off, ln, idx), want):
        assert np.array_equal(g.cpu().numpy(), w)
    live = want[2] >= 0
    for g, w in zip((Ks, Vs), want[3:5]):
        g = gen.to_host_f32(g)
        assert np.array_equal(g[live], w[live]) and (g[~live] == (0.0 if zeroed else 7.0)).all()


@pytest.mark.parametrize("S,N,B", [(1, 700, 16), (2, 5000, 64), (1, 20000, 96)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_centroids_from_ids(saap, S, N, B, dtype):
    g = torch.Generator(device=DEV).manual_seed(B)
    x = torch.randn(S, 2, N, 128, generator=g, device=DEV).to(gen.torch_dtype(dtype))
    cent = torch.randn(2, B, 128, generator=g, device=DEV).to(gen.torch_dtype(dtype))
    ids = torch.randint(0, B - 1, (S, 2, N), generator=g, device=DEV, dtype=torch.int32)      # the last bucket is empty
    off, ln, _, xs, _ = saap.build_bucket_index(ids, x, x, B, 0)
    for normalize in (True, False):
        want = saap.update_centroids(xs, off, ln, cent, normalize)
        got = saap.update_centroids_from_ids(x, ids, cent, normalize)
        assert torch.equal(got, want)
        assert torch.equal(got[:, B - 1], cent[:, B - 1])


@pytest.mark.parametrize("N,B,slack,window", [
    (16400, 255, 1, None), (18432, 256, 0, (1, 2047)), (20000, 257, 3, (2, 30)), (17000, 8191, 1, None), (40961, 8192, 0, (1, 2047)),
    (300000, 2, 1, None), (16385, 1024, 70, None), (16385, 1030, 2, None), (20000, 2051, 3, (1, 30)), (150000, 4099, 1, None)])
def test_runs_scanned_by_every_slice(saap, N, B, slack, window):
    """More than one slice, bucket counts around a multiple of a workgroup's threads (four runs each), no multiple of four, several
    rounds of a wave and the largest."""
    S, Hkv = (1, 1) if N > 100000 else (1, 2)
    ids = np.random.default_rng(N + B).integers(0, B, (S, Hkv, N)).astype(np.int32)
    K = torch.zeros(S, Hkv, N, 128, dtype=torch.bfloat16, device=DEV)
    hK = np.zeros((S, Hkv, N, 128), np.float32)
    d_ids = torch.from_numpy(ids).to(DEV)
    if window:
        got, want = saap.build_windowed_index(d_ids, K, K, B, slack, *window), ref.build_windowed_index(ids, hK, hK, B, slack, *window)
    else:
        got, want = saap.build_bucket_index(d_ids, K, K, B, slack), ref.build_bucket_index(ids, hK, hK, B, slack)
    for g, w in zip(got[:3], want[:3]):
        assert np.array_equal(g.cpu().numpy(), w)
