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
