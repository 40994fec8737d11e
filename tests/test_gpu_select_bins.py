"""Selection from logits where its one-histogram way can go wrong: flat and peaked rows, rows of equal logits, lists around the
candidate buffer, every number of heads, no number among the logits.  The list has to be the oracle's from the probabilities that
the call reports, whichever way it went."""
import numpy as np
import pytest
import torch

from oracle import ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def saap():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the -m gpu tests need a real device")
    import paper_2502_08246_amd as lib
    lib.load_library()
    return lib


@pytest.mark.parametrize("heads", [1, 2, 4, 8])
@pytest.mark.parametrize("B,nprobe", [(16, 1), (64, 8), (144, 2), (1000, 51), (1024, 128), (2048, 129), (4096, 205), (4096, 385),
                                      (4096, 1024), (8192, 1000), (8192, 1025),
                                      (512, 250)])
@pytest.mark.parametrize("spread", [0.0, 0.01, 1.0, 40.0])
def test_lists_from_logits(saap, heads, B, nprobe, spread):
    Hkv = 2
    g = torch.Generator(device=DEV).manual_seed(B + nprobe + heads)
    logits = spread * torch.randn(2, Hkv * heads, B, generator=g, device=DEV)
    logits[1, :, ::3] = logits[1, :, :1]                     # a third of the buckets alike in every head
    probs = torch.empty_like(logits)
    sel = saap.select_buckets_from_logits(logits, Hkv, nprobe, probs=probs)
    assert np.array_equal(sel.cpu().numpy(), ref.select_buckets(probs.cpu().numpy(), Hkv, nprobe))
    # a row's sum of exponentials: trees of at most 8 + 6 + 4 additions, hardware exponentials of 2^-21 on arguments up to 160
    want = torch.softmax(logits.double(), -1)
    assert torch.allclose(probs.double(), want, rtol=2e-4, atol=1e-12)
    assert torch.equal(saap.select_buckets_from_logits(logits, Hkv, nprobe), sel)


def test_a_row_without_numbers_leaves_the_other_lists(saap):
    logits = torch.randn(3, 8, 1024, generator=torch.Generator(device=DEV).manual_seed(1), device=DEV)
    want = saap.select_buckets_from_logits(logits, 2, 51)
    logits[1, 5, 77] = float("nan")
    got = saap.select_buckets_from_logits(logits, 2, 51)
    assert torch.equal(got[0], want[0]) and torch.equal(got[2], want[2]) and torch.equal(got[1, 0], want[1, 0])
    assert ((got >= 0) & (got < 1024)).all()
