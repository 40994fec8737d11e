"""The training products that run as sums of bfloat16 products: lengths of k around the slices, and values that the split does
not hold."""
import pytest
import torch

from test_gpu_train import DEV, problem, to_dev
from test_gpu_train import saap  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


def reference(x, T, params):
    ps = [p.double().requires_grad_() for p in params]
    want = []
    for w in range(x.shape[0]):
        z = torch.relu(x[w].double() @ ps[0][w].T + ps[1][w]) @ ps[2][w].T + ps[3][w]
        t = T[w].double()
        want.append(torch.where(t > 0, t * (t.clamp_min(1e-300).log() - torch.log_softmax(z, -1)), 0 * z).sum(-1).mean())
    want = torch.stack(want)
    want.sum().backward()
    return want.detach(), [p.grad for p in ps]


@pytest.mark.parametrize("R", [32, 33, 47, 48, 49, 64, 65])
@pytest.mark.parametrize("hidden,B", [(256, 260), (255, 261)])
def test_lengths_of_k(saap, R, hidden, B):  # noqa: F811
    """The weight gradients sum over R: one slice of 16 and a second that overlaps it, odd and even numbers of slices.  fp32 sums of
    at most 261 terms in chains of a slice: at most 6.9e-7 here, 2.4e-6 to 2.9e-6 with a pair of planes left out: 1e-6."""
    x, T, params = problem(R, 16, R, 16, hidden, B, torch.float32)
    x, T, params = x.to(DEV), T.to(DEV), to_dev(params)
    loss, grads = saap.query_model_loss_grads(x, T, params)
    want, ref = reference(x, T, params)
    torch.testing.assert_close(loss.double(), want, rtol=1e-5, atol=0.0)
    for name, got, g in zip(("dW1", "db1", "dW2", "db2"), grads, ref):
        dims = tuple(range(1, got.dim()))
        assert ((got.double() - g).norm(dim=dims) <= 1e-6 * g.norm(dim=dims)).all(), name


# Values whose planes are named: 8 bits, what half a last bit of those leaves room for, and the same again.
H0, H1, H2 = 4096.0, 4.0, 2.0 ** -8


def columns_of(pair, c):
    """Hidden units and their output weights, for which every pair of planes but this one cancels: logits c."""
    one = torch.ones_like(c)
    return {
        (0, 1): ([256.0, 256.0], [H0 + c / 256, -H0 * one]),
        (1, 0): ([H0 + H1, H0], [c / H1, -c / H1]),
        (1, 1): ([512.0 + 1, 512.0, 512.0 + 1, 512.0], [H0 + c, -H0 - c, -H0 * one, H0 * one]),
        (0, 2): ([256.0, 256.0], [H0 + 5 + c / 256, -(H0 + 5) * one]),
        (2, 0): ([H0 + H1 + H2, H0 + H1], [c / H2, -c / H2]),
    }[pair]


@pytest.mark.parametrize("pair", [(0, 1), (1, 0), (1, 1), (0, 2), (2, 0)])
@pytest.mark.parametrize("R", [128, 512])
def test_every_pair_of_planes(saap, pair, R):  # noqa: F811
    """Logits that one pair of planes alone makes (plane of h, plane of W2): without it they are 0.  Every product and sum is exact, so
    the loss and db2 are as far off as the softmax of given logits: hardware exponentials of 2^-21, sums of 1024."""
    Hw, d, hidden, B = 16, 16, 64, 1024
    c = torch.randint(-30, 31, (Hw, B), generator=torch.Generator().manual_seed(R)).float() / 8
    units, weights = columns_of(pair, c)
    x, T, (W1, b1, W2, b2) = problem(R, Hw, R, d, hidden, B, torch.float32)
    W1, b1, W2, b2 = 0 * W1, 0 * b1 - 1, 0 * W2, 0 * b2
    for k, (h, w) in enumerate(zip(units, weights)):
        b1[:, 7 * k + 3], W2[:, :, 7 * k + 3] = h, w
    assert torch.equal(W2.double() @ b1.clamp_min(0).double().unsqueeze(2), c.double().unsqueeze(2)), "logits"
    x, T, params = x.to(DEV), T.to(DEV), to_dev((W1, b1, W2, b2))
    loss, grads = saap.query_model_loss_grads(x, T, params)
    want, ref = reference(x, T, params)
    torch.testing.assert_close(loss.double(), want, rtol=1e-5, atol=0.0)
    assert ((grads[3].double() - ref[3]).norm(dim=1) <= 3e-6 * ref[3].norm(dim=1)).all()


@pytest.mark.parametrize("R,hidden,B", [(512, 256, 512), (129, 256, 512)])
def test_values_beyond_bfloat16(saap, R, hidden, B):  # noqa: F811
    """A unit that no row turns on, with output weights that round to infinity in bfloat16: they add nothing, as in fp32."""
    Hw, d, off = 16, 32, 5
    x, T, (W1, b1, W2, b2) = problem(3, Hw, R, d, hidden, B, torch.float32)
    b1[:, off], W2[:, :, off] = -1e4, 0.0
    x, T, params = x.to(DEV), T.to(DEV), to_dev((W1, b1, W2, b2))
    huge = tuple(p.clone() for p in params)
    huge[2][:, :, off] = 3.4e38
    assert torch.isfinite(huge[2]).all() and torch.isinf(huge[2].to(torch.bfloat16)).any()
    want, ref = reference(x, T, params)
    loss, grads = saap.query_model_loss_grads(x, T, huge)
    torch.testing.assert_close(loss.double(), want, rtol=1e-5, atol=0.0)
    for name, got, g in zip(("dW1", "db1", "dW2", "db2"), grads, ref):
        assert ((got.double() - g).norm() <= 3e-6 * g.norm()), name


# dz follows the scale of T, h and the second operand of dW1 that of x, da that of W2.  The third is the same problem with no value
# near an end of the range.
@pytest.mark.parametrize("Hw,R,hidden,B", [(16, 320, 512, 512), (16, 640, 512, 1024)])
@pytest.mark.parametrize("scales,plain,tol", [
    ((0, -100, 0), (0, 0, 0), 1e-7), ((-118, 20, 0), (-70, 20, 0), 1e-7), ((0, 20, -118), (0, 20, -70), 1e-7),
    ((0, 100, 0), (0, 0, 0), 2e-6)])
def test_products_of_operands_of_any_size(saap, Hw, R, hidden, B, scales, plain, tol):  # noqa: F811
    """Powers of two on x, T and W2 (with W2 or h below 2^-60 the logits are b2): the gradients are the plain problem's times powers
    of two.  Down to 2^-126 that is exact, and the few values below it are off by 2^-32 of the others: 1e-7.  Sums beyond 2^80 are made
    with fp32 instructions: as far apart as the two ways are (6e-7 and 4e-7 from float64, twice that)."""
    x, T, (W1, b1, W2, b2) = problem(11, Hw, R, 128, hidden, B, torch.float32)

    def gradients(ex, eT, eW):
        params = to_dev((W1, 0 * b1, W2 * 2.0 ** eW, b2))
        return [g.double() for g in saap.query_model_loss_grads((x * 2.0 ** ex).to(DEV), (T * 2.0 ** eT).to(DEV), params)[1]]

    (ex, eT, eW), got, want = (s - p for s, p in zip(scales, plain)), gradients(*scales), gradients(*plain)
    for name, g, w, e in zip(("dW1", "db1", "dW2", "db2"), got, want, (ex + eT + eW, eT + eW, ex + eT, eT)):
        w = w * 2.0 ** e
        dims = tuple(range(1, w.dim()))
        assert (w.norm(dim=dims) > 0).all() and ((g - w).norm(dim=dims) <= tol * w.norm(dim=dims)).all(), name


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_a_weight_that_is_no_number_spoils_its_set_only(saap, bad):  # noqa: F811
    x, T, params = problem(4, 16, 256, 32, 256, 512, torch.float32)
    x, T, params = x.to(DEV), T.to(DEV), to_dev(params)
    broken = tuple(p.clone() for p in params)
    broken[2][3, 7, 9] = bad
    want_loss, want = saap.query_model_loss_grads(x, T, params)
    loss, grads = saap.query_model_loss_grads(x, T, broken)
    assert loss[3].isnan()
    others = torch.arange(16, device=DEV) != 3
    assert torch.equal(loss[others], want_loss[others])
    for name, got, g in zip(("dW1", "db1", "dW2", "db2"), grads, want):
        assert torch.equal(got[others], g[others]), name
        assert got[3].isnan().any(), name
