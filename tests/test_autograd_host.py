"""What autograd records of the CP loss's backward pass, with the library's calls replaced
by torch on the CPU."""
import pytest

torch = pytest.importorskip("torch")

from paper_2507_15121_amd import api, autograd  # noqa: E402
from paper_2507_15121_amd.autograd import sparse_cp_loss  # noqa: E402


class _Coo:
    """A sparse tensor and the loss's calls on it."""

    def __init__(self, dims, nnz, seed=0):
        g = torch.Generator().manual_seed(seed)
        self.dims = dims
        self.idx = [torch.randint(d, (nnz,), generator=g) for d in dims]
        self.val = torch.rand(nnz, generator=g, dtype=torch.float64)

    def residuals(self, factors):
        p = 1.0
        for i, f in zip(self.idx, factors):
            p = p * f.double()[i]
        return self.val - p.sum(1)

    def grad(self, mode, factors, scale):
        p = self.residuals(factors)[:, None]
        for w, (i, f) in enumerate(zip(self.idx, factors)):
            if w != mode:
                p = p * f.double()[i]
        out = torch.zeros(self.dims[mode], factors[0].shape[1], dtype=torch.float64)
        return (scale * out.index_add(0, self.idx[mode], p)).float()


@pytest.fixture
def on_cpu(monkeypatch):
    monkeypatch.setattr(api, "cp_loss", lambda t, f: t.residuals(f).square().sum())
    monkeypatch.setattr(api, "cp_loss_grad", lambda t, d, f, s: (t.residuals(f).square().sum(), t.grad(d, f, s)))
    monkeypatch.setattr(api, "cp_grad_scaled", lambda t, d, f, s, x: t.grad(d, f, s * float(x)))
    monkeypatch.setattr(api, "scale_", lambda x, s: x.mul_(s))
    assert autograd.api is api


def _factors(dims, rank, need):
    g = torch.Generator().manual_seed(1)
    return [torch.rand(d, rank, generator=g).requires_grad_(n) for d, n in zip(dims, need)]


def test_gradients(on_cpu):
    t = _Coo((7, 6, 5), 60)
    F = _factors(t.dims, 4, (True, False, True))
    (3.0 * sparse_cp_loss(t, *F)).backward()
    for d in (0, 2):
        torch.testing.assert_close(F[d].grad, 3.0 * t.grad(d, [f.detach() for f in F], -2.0))
    assert F[1].grad is None


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_graph_through_the_upstream_gradient(on_cpu, mode):
    """create_graph=True: the gradient that the forward pass made is linear in dL_out, and
    a second pass finds that derivative (a learned weight of the loss, say)."""
    t = _Coo((7, 6, 5), 60)
    F = _factors(t.dims, 4, [d == mode for d in range(3)])
    w = torch.tensor(1.5, dtype=torch.float64, requires_grad=True)
    g, = torch.autograd.grad(w * sparse_cp_loss(t, *F), F[mode], create_graph=True)
    base = t.grad(mode, [f.detach() for f in F], -2.0)
    torch.testing.assert_close(g.detach(), 1.5 * base)
    x = torch.rand_like(base)
    (g * x).sum().backward()
    torch.testing.assert_close(w.grad, (base.double() * x.double()).sum(), rtol=1e-5, atol=1e-5)
