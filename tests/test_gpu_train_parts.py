"""The training products whose k several groups of waves share out, and those of the widest tiles: lengths of k that leave a group
without a slice, short first slices, rows that start on 16 bytes and rows that do not, values that are no numbers in any group."""
import pytest
import torch

from test_gpu_train import DEV, problem, to_dev
from test_gpu_train import saap  # noqa: F401  (the fixture)
from test_gpu_train_planes import reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hw,R,hidden,B", [
    (16, 140, 136, 200), (16, 141, 135, 201), (16, 128, 129, 224), (16, 143, 145, 223),      # four groups
    (18, 100, 72, 300), (18, 101, 65, 301), (16, 300, 200, 260), (16, 301, 201, 259),        # two
    (16, 1100, 64, 300), (16, 1030, 66, 65),                                                 # 128 x 64
    (16, 520, 260, 516), (16, 513, 257, 513),                                                # 128 x 128, edges
])
def test_shared_k(saap, Hw, R, hidden, B):  # noqa: F811
    """fp32 sums of at most 1100 terms in chains of a slice: at most 1e-6 (6e-7 measured for the products of one group)."""
    x, T, params = problem(R + B, Hw, R, 24, hidden, B, torch.float32)
    x, T, params = x.to(DEV), T.to(DEV), to_dev(params)
    loss, grads = saap.query_model_loss_grads(x, T, params)
    again = saap.query_model_loss_grads(x, T, params)[1]
    want, ref = reference(x, T, params)
    torch.testing.assert_close(loss.double(), want, rtol=1e-5, atol=0.0)
    for name, got, g, rep in zip(("dW1", "db1", "dW2", "db2"), grads, ref, again):
        dims = tuple(range(1, got.dim()))
        assert ((got.double() - g).norm(dim=dims) <= 1e-6 * g.norm(dim=dims)).all(), name
        assert torch.equal(got, rep), name


@pytest.mark.parametrize("unit", [0, 40, 80, 135])
def test_huge_weight_in_any_group(saap, unit):  # noqa: F811
    """Output weights that round to infinity in bfloat16, of a unit that no row turns on, in each of the four groups of k."""
    Hw, R, hidden, B = 16, 140, 136, 200
    x, T, (W1, b1, W2, b2) = problem(3, Hw, R, 32, hidden, B, torch.float32)
    b1[:, unit], W2[:, :, unit] = -1e4, 0.0
    x, T, params = x.to(DEV), T.to(DEV), to_dev((W1, b1, W2, b2))
    huge = tuple(p.clone() for p in params)
    huge[2][5, :, unit] = 3.4e38
    want, ref = reference(x, T, params)
    loss, grads = saap.query_model_loss_grads(x, T, huge)
    torch.testing.assert_close(loss.double(), want, rtol=1e-5, atol=0.0)
    for name, got, g in zip(("dW1", "db1", "dW2", "db2"), grads, ref):
        assert ((got.double() - g).norm() <= 3e-6 * g.norm()), name


@pytest.mark.parametrize("Hw,R,d,hidden,B", [
    (16, 129, 128, 256, 40), (16, 131, 129, 254, 33),      # dW1 in four groups
    (16, 70, 200, 512, 40), (16, 67, 201, 500, 40),        # two
    (16, 40, 512, 320, 40), (32, 36, 256, 512, 40), (32, 35, 64, 2048, 40),      # one, 128 x 128, 128 x 64
    (2, 20, 12, 20, 24), (3, 33, 13, 30, 25), (8, 1000, 128, 512, 64),           # few tiles; the first product's large ones
])
def test_features_in_bfloat16(saap, Hw, R, d, hidden, B):  # noqa: F811
    """Against the same features in fp32, whose values are the same: all but dW1 bit for bit, and dW1 as far off as fp32 sums of R
    terms in another order may be (4e-7 from float64 each: 1e-6)."""
    x, T, params = problem(R + d, Hw, R, d, hidden, B, torch.bfloat16)
    x, T, params = x.to(torch.bfloat16).to(DEV), T.to(DEV), to_dev(params)
    loss, grads = saap.query_model_loss_grads(x, T, params)
    want_loss, want = saap.query_model_loss_grads(x.float(), T, params)
    assert torch.equal(loss, want_loss)
    for name, got, g in zip(("dW1", "db1", "dW2", "db2"), grads, want):
        dims = tuple(range(1, got.dim()))
        assert ((got - g).norm(dim=dims) <= 1e-6 * g.norm(dim=dims)).all() if name == "dW1" else torch.equal(got, g), name
