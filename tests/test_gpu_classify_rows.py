"""The classifier at row counts around the switch to the row-tiled output kernel and its tile edges, with hidden widths
and bucket counts that leave partial chunks and tiles, and in fp32 with every division of the hidden units among the
waves, against the oracle."""
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


@pytest.mark.parametrize("S,Hq,Hkv,Hw,hidden,B,dtype", [
    (63, 1, 1, 1, 32, 16, "bf16"), (64, 1, 1, 1, 32, 16, "bf16"), (13, 10, 2, 2, 96, 48, "bf16"), (16, 8, 2, 2, 64, 208, "bf16"),
    (65, 3, 1, 3, 160, 80, "bf16"), (32, 32, 8, 8, 512, 1008, "bf16"), (43, 6, 2, 1, 224, 1040, "bf16"), (257, 4, 4, 1, 544, 2064, "bf16"),
    (1, 1, 1, 1, 32, 16, "f32"), (2, 4, 2, 2, 96, 48, "f32"), (5, 4, 1, 1, 160, 80, "f32"), (1, 2, 2, 2, 544, 64, "f32")])
def test_logits(saap, S, Hq, Hkv, Hw, hidden, B, dtype):
    g = torch.Generator(device=DEV).manual_seed(S * 131 + hidden)
    dt = gen.torch_dtype(dtype)
    randn = lambda *s: torch.randn(*s, generator=g, device=DEV)  # noqa: E731
    xq = (2 * randn(S, Hq, 128)).to(dt)
    W1, W2 = (randn(Hw, hidden, 128) / 128 ** 0.5).to(dt), (randn(Hw, B, hidden) / hidden ** 0.5).to(dt)
    b1, b2 = randn(Hw, hidden), randn(Hw, B)
    h = gen.to_host_f32
    for biases in ((b1, b2), (None, None)):
        got = saap.classify_queries(xq, W1, biases[0], W2, biases[1], Hkv, output_kind=saap.LOGITS)
        hb = [np.zeros(t.shape, np.float32) if b is None else h(b) for b, t in zip(biases, (b1, b2))]
        want = ref.classify_queries(h(xq), h(W1), hb[0], h(W2), hb[1], Hkv, output_kind=1)
        np.testing.assert_allclose(h(got), want, rtol=2e-5, atol=5e-5)


@pytest.mark.parametrize("hidden", [32, 64, 96, 544])
def test_an_infinite_weight_counts_once(saap, hidden):
    """A weight of the last hidden unit, which partial chunks read again: fp32 against float64, and many bf16 rows against the
    same rows a few at a time."""
    g = torch.Generator(device=DEV).manual_seed(hidden)
    randn = lambda *s: torch.randn(*s, generator=g, device=DEV)  # noqa: E731
    S, B = 80, 32
    xq, W1, W2, b1 = randn(S, 1, 128), randn(1, hidden, 128) / 128 ** 0.5, randn(1, B, hidden), randn(1, hidden)
    b1[0, -1] = 100.0                                     # the unit is above zero for every row
    W2[0, 3, -1], W2[0, 17, -1] = float("inf"), -float("inf")
    got = saap.classify_queries(xq, W1, b1, W2, None, 1, output_kind=saap.LOGITS)[:, 0].cpu()
    want = (xq[:, 0].double() @ W1[0].double().T + b1[0].double()).clamp_min(0).cpu() @ W2[0].double().cpu().T
    assert torch.isinf(want).sum() == 2 * S
    torch.testing.assert_close(got.double(), want, rtol=2e-5, atol=5e-5 * hidden ** 0.5)      # weights of magnitude 1, not 1 / sqrt(hidden)
    x16, W1h, W2h = (t.bfloat16() for t in (xq, W1, W2))
    many = saap.classify_queries(x16, W1h, b1, W2h, None, 1, output_kind=saap.LOGITS)
    few = torch.cat([saap.classify_queries(x16[i:i + 16], W1h, b1, W2h, None, 1, output_kind=saap.LOGITS) for i in range(0, S, 16)])
    assert torch.isinf(few).any()
    torch.testing.assert_close(many, few, rtol=2e-5, atol=5e-5 * hidden ** 0.5, equal_nan=True)
