"""Index builds at the sizes where the sort changes its shape (one launch for short contexts, slices beyond) and at the
edges of its rounds and slices, zeroed free slots included, against the oracle; the centroid step from bucket ids
against the one from grouped features, bit for bit."""
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
    # most keys in a few buckets, some buckets empty, a few ids outside the range (dropped)
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
