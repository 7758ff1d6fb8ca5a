"""The differentiable expectation value against a dense contraction of the
whole state vector, and its gradients against finite differences (float64,
central differences of step 1e-6 on values of order one: gradcheck's defaults)."""
import pytest
import torch

from paper_1504_00992_amd import gradient


def _chain(n, d, cap, seed):
    gen = torch.Generator().manual_seed(seed)
    chi = [1] + [min(cap, d ** min(k + 1, n - 1 - k)) for k in range(n - 1)] + [1]
    gamma = torch.zeros((n, d, cap, cap), dtype=torch.complex128)
    lam = torch.zeros((n - 1, cap), dtype=torch.float64)
    for k in range(n):
        gamma[k, :, :chi[k], :chi[k + 1]] = torch.randn(
            (d, chi[k], chi[k + 1]), generator=gen, dtype=torch.complex128)
    for k in range(n - 1):
        lam[k, :chi[k + 1]] = torch.rand(chi[k + 1], generator=gen, dtype=torch.float64) + 0.1
    op = torch.randn((d, d), generator=gen, dtype=torch.complex128)
    return gamma, lam, op + op.mH


def _dense(gamma, lam, op, site):
    n, d = gamma.shape[0], gamma.shape[1]
    psi = gamma[0, :, 0, :]                                   # (i1, c)
    for k in range(1, n):
        psi = torch.tensordot(psi * lam[k - 1], gamma[k].permute(1, 0, 2), 1).flatten(0, 1)
    psi = psi[:, 0].reshape([d] * n)
    opsi = psi if not 0 <= site < n else torch.movedim(
        torch.tensordot(op, psi, ([1], [site])), 0, site)
    return (torch.sum(psi.conj() * opsi) / torch.sum(psi.conj() * psi)).real


@pytest.mark.parametrize("n,d,cap", [(1, 2, 1), (2, 2, 2), (5, 2, 4), (4, 3, 7), (6, 2, 3)])
def test_against_the_dense_state(n, d, cap):
    gamma, lam, op = _chain(n, d, cap, n * 10 + d)
    for site in range(-1, n + 1):
        got = gradient.expectation(gamma, lam, op, site)
        assert abs(got - _dense(gamma, lam, op, site)) <= 1e-12 * max(1.0, op.abs().sum())


def test_gradients():
    gamma, lam, op = _chain(4, 2, 3, 8)
    gamma.requires_grad_(True)
    lam.requires_grad_(True)
    for site in (0, 2, 3):
        assert torch.autograd.gradcheck(lambda g, l: gradient.expectation(g, l, op, site), (gamma, lam))
