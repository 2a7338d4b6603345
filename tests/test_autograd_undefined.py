"""The reverse pass of autograd.poly_eval when no adjoint reaches the value: the
operation after it returns none.  The gradients are those of a zero adjoint, not
absent (no GPU needed: the polynomial's device calls are replaced by plain ones)."""
import types

import torch

from paper_2101_10881_amd import mdpe
from paper_2101_10881_amd.autograd import poly_eval


def _scaling_polynomial(m, n, N, d, seen):
    """A Polynomial whose value is a_0 and whose reverse pass returns its adjoint, spread over the inputs."""
    P = mdpe.Polynomial.__new__(mdpe.Polynomial)
    P.plan = types.SimpleNamespace(info={"flags": mdpe.MDPE_KEEP_MONOMIAL_VALUES})
    P.m, P.n, P.N, P.d = m, n, N, d
    P.new_workspace = lambda: torch.empty(1)
    P.eval_and_diff = lambda c, z, workspace: (c[:, 0].clone(), torch.zeros(m, n, d + 1, dtype=c.dtype))

    def adjoint(ybar, grad, workspace):
        seen.append(ybar)
        return ybar[:, None].expand(m, N + 1, d + 1).clone(), ybar[:, None].expand(m, n, d + 1).clone()
    P.adjoint = adjoint
    return P


class _NoGradient(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x):
        return x.clone()

    @staticmethod
    def backward(ctx, g):
        return None


def _inputs(m=2, n=3, N=4, d=5):
    c = torch.ones(m, N + 1, d + 1, dtype=torch.float64, requires_grad=True)
    z = torch.ones(m, n, d + 1, dtype=torch.float64, requires_grad=True)
    return c, z, (m, n, N, d)


def test_undefined_adjoint_gives_zero_gradients():
    c, z, shape = _inputs()
    seen = []
    value, _ = poly_eval(c, z, _scaling_polynomial(*shape, seen))
    cbar, zbar = torch.autograd.grad(_NoGradient.apply(value).sum(), (c, z))
    assert cbar.shape == c.shape and not cbar.any()
    assert zbar.shape == z.shape and not zbar.any()
    assert seen[0].shape == value.shape and seen[0].dtype == value.dtype


def test_defined_adjoint_passes_unchanged():
    c, z, shape = _inputs()
    seen = []
    value, _ = poly_eval(c, z, _scaling_polynomial(*shape, seen))
    ybar = torch.arange(12, dtype=torch.float64).reshape(2, 6)
    cbar, _ = torch.autograd.grad(value, (c, z), ybar)
    assert torch.equal(seen[0], ybar) and torch.equal(cbar[:, 3], ybar)
