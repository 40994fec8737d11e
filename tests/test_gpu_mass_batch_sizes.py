"""bucket_attention_mass_batch at the edges of its query tiles and key tiles, with empty buckets, with a negative score
scale and one of zero, and with scores so far apart that the reference of the running sums has to move, against float64 numpy."""
import numpy as np
import pytest
import torch

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


@pytest.mark.parametrize("R,lens,scale,spread", [
    (1, [1], 0.09, 1.0), (31, [0, 1, 31, 32, 33, 0, 65, 2], 0.09, 1.0), (128, [64] * 5, 0.09, 1.0), (129, [3, 0, 40] * 30, 0.09, 1.0),
    (256, [33, 95, 1, 0], -0.09, 1.0), (300, [10, 200, 31], 0.09, 40.0), (257, [70, 0, 5, 64, 90], -0.09, 40.0),
    (40, [1, 0, 2] * 400, 0.09, 1.0), (130, [0, 0, 0], 0.09, 1.0),
    (129, [3, 0, 32, 40], 0.0, 1.0), (256, [33, 95, 1, 64], -0.0, 1.0), (40, [33, 5, 64], 1e-40, 1.0)])
def test_mass(saap, R, lens, scale, spread):
    Hkv, B, N = 2, len(lens), max(sum(lens), 1)
    g = torch.Generator(device=DEV).manual_seed(R)
    q = torch.randn(1, Hkv, R, 128, generator=g, device=DEV).to(torch.bfloat16)
    # later keys reach far above earlier ones when `spread` is large (score range of some hundred bits)
    grow = torch.linspace(1.0, spread, N, device=DEV).view(1, 1, N, 1)
    K = (grow * torch.randn(1, Hkv, N, 128, generator=g, device=DEV)).to(torch.bfloat16)
    off = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device=DEV).view(1, 1, B + 1).repeat(1, Hkv, 1).contiguous()
    ln = torch.tensor(lens, dtype=torch.int32, device=DEV).view(1, 1, B).repeat(1, Hkv, 1).contiguous()
    mass, lse = saap.bucket_attention_mass_batch(q, K, off, ln, scale)
    mass, lse = mass.cpu().numpy(), lse.cpu().numpy()
    hq, hK = gen.to_host_f32(q).astype(np.float64), gen.to_host_f32(K).astype(np.float64)
    for h in range(Hkv):
        if sum(lens) == 0:
            assert not mass[0, h].any() and np.isneginf(lse[0, h]).all()
            continue
        t = scale * hq[0, h] @ hK[0, h].T
        top = t.max(-1, keepdims=True)
        w = np.exp(t - top)
        want = np.stack([w[:, a:a + n].sum(-1) for a, n in zip(np.cumsum([0] + list(lens))[:-1], lens)], -1)
        total = w.sum(-1, keepdims=True)
        # an fp32 score of magnitude s is off by about 2^-24 sqrt(128) s, which the exponential turns into a relative error
        tol = 1e-5 * max(1.0, np.abs(t).max())
        np.testing.assert_allclose(mass[0, h], want / total, rtol=tol, atol=1e-7)
        np.testing.assert_allclose(lse[0, h], (top + np.log(total))[:, 0], rtol=1e-5, atol=1e-4)


@pytest.mark.parametrize("Hkv,R,B", [(2, 200, 1024), (64, 2048, 1024), (64, 512, 8192)])
def test_the_same_inputs_give_the_same_bits(saap, Hkv, R, B):
    """One, 256 and 512 buckets to a workgroup: the running reference goes through them in one order."""
    g = torch.Generator(device=DEV).manual_seed(B)
    N = 4 * B
    ids = torch.randint(0, B, (1, Hkv, N), generator=g, device=DEV, dtype=torch.int32)
    K = 3 * torch.randn(1, Hkv, N, 128, generator=g, device=DEV)
    K *= torch.rand(1, Hkv, N, 1, generator=g, device=DEV) * 4          # the reference moves within a workgroup's buckets
    K = K.to(torch.bfloat16)
    off, ln, _, Ks, _ = saap.build_bucket_index(ids, K, K, B)
    q = torch.randn(1, Hkv, R, 128, generator=g, device=DEV).to(torch.bfloat16)
    mass, lse = saap.bucket_attention_mass_batch(q, Ks, off, ln, 0.09)
    for _ in range(8):
        again, again_lse = saap.bucket_attention_mass_batch(q, Ks, off, ln, 0.09)
        assert torch.equal(mass, again) and torch.equal(lse, again_lse)


@pytest.mark.parametrize("scale", [0.09, -0.09])
def test_an_infinite_score_stays_in_its_bucket(saap, scale):
    """A key with an infinite feature, in a bucket that others of its workgroup follow: as the call for decode steps, which
    takes every bucket by itself, gives it."""
    B, N, R = 600, 24000, 8
    g = torch.Generator(device=DEV).manual_seed(5)
    ids = torch.randint(0, B, (8, 32, N // 8), generator=g, device=DEV, dtype=torch.int32)
    K = torch.randn(8, 32, N // 8, 128, generator=g, device=DEV).to(torch.bfloat16)
    q = torch.randn(8, 32, R, 128, generator=g, device=DEV).to(torch.bfloat16)
    K[0, 0, 100, 7] = K[1, 3, 2000, 9] = float("inf")
    off, ln, _, Ks, _ = saap.build_bucket_index(ids, K, K, B)
    mass, lse = saap.bucket_attention_mass_batch(q, Ks, off, ln, scale)
    want, want_lse = saap.bucket_attention_mass(q.view(8, 32 * R, 128), Ks, off, ln, scale)
    want, want_lse = want.view_as(mass), want_lse.view_as(lse)
    bad = ~torch.isfinite(want)
    assert 0 < bad.sum() <= 2 * R and (lse[0, 0] == -float("inf")).any()
    assert torch.equal(~torch.isfinite(mass), bad) and torch.equal(torch.isinf(lse), torch.isinf(want_lse))
    # scores of magnitude 8 in sums of another order: as in test_mass
    torch.testing.assert_close(mass[~bad], want[~bad], rtol=1e-4, atol=1e-7)


@pytest.mark.parametrize("R,B", [
    (1, 1), (31, 31), (40, 128), (33, 129), (33, 255), (32, 256), (40, 257), (5, 511), (40, 512), (33, 513), (33, 1023), (64, 1024),
    (33, 1025)])
def test_mass_rows_of_odd_lengths(saap, R, B):
    """Rows held in registers (129 to 1024 buckets) and rows read twice: every third bucket empty."""
    test_mass(saap, R, [(2, 0, 3)[b % 3] for b in range(B)], 0.09, 1.0)
