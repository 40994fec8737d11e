"""Loss and gradients of the query model where its matrix products take their large tiles: rows that start on 16 bytes and rows
that do not, reductions that end inside a slice, operands on either side."""
import pytest
import torch

from test_gpu_train import DEV, problem, to_dev
from test_gpu_train import saap  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hw,R,d,hidden,B", [
    (16, 900, 40, 132, 520), (16, 900, 40, 131, 521), (16, 60, 64, 452, 1030), (16, 60, 64, 450, 1032), (8, 1000, 128, 512, 1024),
])
def test_large_products(saap, Hw, R, d, hidden, B):  # noqa: F811
    x, T, params = problem(5, Hw, R, d, hidden, B, torch.float32)
    x, T, params = x.to(DEV), T.to(DEV), to_dev(params)
    loss, grads = saap.query_model_loss_grads(x, T, params)
    again = saap.query_model_loss_grads(x, T, params)[1]
    ps = [p.double().requires_grad_() for p in params]
    want = []
    for w in range(Hw):
        z = torch.relu(x[w].double() @ ps[0][w].T + ps[1][w]) @ ps[2][w].T + ps[3][w]
        t = T[w].double()
        want.append(torch.where(t > 0, t * (t.clamp_min(1e-300).log() - torch.log_softmax(z, -1)), 0 * z).sum(-1).mean())
    want = torch.stack(want)
    want.sum().backward()
    torch.testing.assert_close(loss.double(), want.detach(), rtol=1e-5, atol=0.0)
    for name, got, p, rep in zip(("dW1", "db1", "dW2", "db2"), grads, ps, again):
        err = (got.double() - p.grad).norm(dim=tuple(range(1, got.dim()))) / p.grad.norm(dim=tuple(range(1, got.dim())))
        assert err.max() < 3e-6, (name, err)
        assert torch.equal(got, rep), name


def test_more_rows_than_one_launch_of_small_tiles(saap):  # noqa: F811
    """65535 tiles of 32 rows and 41 rows more, reductions too short for the large tiles.  Only the last 50 rows have a target,
    so that the gradients are sums over those (fp32 sums of 50 terms: 50 * 2^-24 = 3e-6 relative; 1e-5 with the logits' own)."""
    R, live, (d, hidden, B) = 65535 * 32 + 41, 50, (4, 8, 8)
    x, T, params = problem(7, 1, live, d, hidden, B, torch.float32)
    params = to_dev(params)
    X, target = torch.zeros(1, R, d, device=DEV), torch.zeros(1, R, B, device=DEV)
    X[:, -live:], target[:, -live:] = x.to(DEV), T.to(DEV)
    loss, grads = saap.query_model_loss_grads(X, target, params)
    ps = [p.double().requires_grad_() for p in params]
    z = torch.relu(X[0, -live:].double() @ ps[0][0].T + ps[1][0]) @ ps[2][0].T + ps[3][0]
    t = target[0, -live:].double()
    want = torch.where(t > 0, t * (t.clamp_min(1e-300).log() - torch.log_softmax(z, -1)), 0 * z).sum() / R
    want.backward()
    torch.testing.assert_close(loss[0].double(), want.detach(), rtol=1e-5, atol=0.0)
    for name, got, p in zip(("dW1", "db1", "dW2", "db2"), grads, ps):
        assert (got.double() - p.grad).norm() <= 1e-5 * p.grad.norm(), name


@pytest.mark.parametrize("B", [1, 255, 257, 1023, 1025, 2047, 2048, 2049])
def test_rows_held_and_rows_read_again(saap, B):  # noqa: F811
    """Row lengths around what a workgroup holds; fp32 sums of up to 2049 terms in trees of at most 16 + 8 additions, hardware
    exponentials and logarithms of 2^-21 or so on arguments around 10: 1e-5."""
    R, d, hidden = 37, 24, 16
    x, T, params = problem(B, 2, R, d, hidden, B, torch.float32)
    T = T.nan_to_num(0.0) if B > 1 else torch.ones_like(T) * (torch.arange(R)[None, :, None] % 2)
    x, T, params = x.to(DEV), T.to(DEV), to_dev(params)
    loss, grads = saap.query_model_loss_grads(x, T, params)
    ps = [p.double().requires_grad_() for p in params]
    want = []
    for w in range(2):
        z = torch.relu(x[w].double() @ ps[0][w].T + ps[1][w]) @ ps[2][w].T + ps[3][w]
        t = T[w].double()
        want.append(torch.where(t > 0, t * (t.clamp_min(1e-300).log() - torch.log_softmax(z, -1)), 0 * z).sum(-1).mean())
    torch.stack(want).sum().backward()
    torch.testing.assert_close(loss.double(), torch.stack(want).detach(), rtol=1e-5, atol=1e-6)
    for name, got, p in zip(("dW1", "db1", "dW2", "db2"), grads, ps):
        assert (got.double() - p.grad).norm() <= 1e-5 * p.grad.norm() + 1e-6, name
