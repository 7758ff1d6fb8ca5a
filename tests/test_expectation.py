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


def _by_einsum(gamma, lam, op, site):
    """The definition, one environment at a time."""
    n, cap = gamma.shape[0], gamma.shape[-1]
    op = torch.as_tensor(op, dtype=torch.complex128)
    envs = []
    for with_op in (True, False):
        env = torch.zeros((cap, cap), dtype=torch.complex128)
        env[0, 0] = 1.0
        for k in range(n):
            a = gamma[k] * lam[k].to(torch.complex128)[None, None, :] if k < n - 1 else gamma[k]
            if with_op and k == site:
                env = torch.einsum("ab,iac,ij,jbd->cd", env, a.conj(), op, a)
            else:
                env = torch.einsum("ab,iac,ibd->cd", env, a.conj(), a)
        envs.append(env[0, 0])
    return (envs[0] / envs[1]).real


_FORMS = {
    "op 1 x 1": lambda g, l, o: (g, l, o[:1, :1]),
    "op 1 x d": lambda g, l, o: (g, l, o[:1]),
    "op d x 1": lambda g, l, o: (g, l, o[:, :1]),
    "op [1, d, d]": lambda g, l, o: (g, l, o[None]),
    "op of rank 1": lambda g, l, o: (g, l, o[0]),
    "op of rank 0": lambda g, l, o: (g, l, o[0, 0]),
    "op too small": lambda g, l, o: (g, l, o[:2, :2]),
    "op real list": lambda g, l, o: (g, l, o.real.tolist()),
    "one local state": lambda g, l, o: (g[:, :1], l, o),
    "lam one row": lambda g, l, o: (g, l[:1], o),
    "lam short": lambda g, l, o: (g, l[:-1], o),
    "lam a row more": lambda g, l, o: (g, torch.cat([l, l[:1]]), o),
    "lam one column": lambda g, l, o: (g, l[:, :1], o),
    "lam of rank 1": lambda g, l, o: (g, l[:, 0], o),
    "lam of rank 3": lambda g, l, o: (g, l[:, None], o),
    "lam a list": lambda g, l, o: (g, list(l), o),
    "lam a short list": lambda g, l, o: (g, list(l)[:2], o),
    "lam float32": lambda g, l, o: (g, l.float(), o),
    "lam complex": lambda g, l, o: (g, l.to(torch.complex128), o),
    "lam integer": lambda g, l, o: (g, (10 * l).long(), o),
    "one site, no lam": lambda g, l, o: (g[:1], None, o),
    "gamma complex64": lambda g, l, o: (g.to(torch.complex64), l, o),
    "gamma real": lambda g, l, o: (g.real, l, o),
    "gamma transposed": lambda g, l, o: (g.transpose(-1, -2), l, o),
    "gamma expanded": lambda g, l, o: (g[:1].expand_as(g), l, o),
    "gamma not square": lambda g, l, o: (g[..., :3, :], l, o),
    "gamma of rank 5": lambda g, l, o: (g[:1, None, :1], l, o[:1, :1]),
}


@pytest.mark.parametrize("form", _FORMS)
def test_forms_taken_and_refused(form):
    # what the definition takes is taken, with its value, and what it refuses is
    # refused with the same kind of error
    gen = torch.Generator().manual_seed(3)
    gamma = torch.randn((5, 3, 4, 4), generator=gen, dtype=torch.complex128)
    lam = torch.rand((4, 4), generator=gen, dtype=torch.float64) + 0.1
    op = torch.randn((3, 3), generator=gen, dtype=torch.complex128)
    args = _FORMS[form](gamma, lam, op + op.mH)
    for site in (0, 2, 9):
        try:
            want = _by_einsum(*args, site)
        except (RuntimeError, IndexError) as e:
            with pytest.raises(type(e)):
                gradient.expectation(*args, site)
        else:
            assert abs(gradient.expectation(*args, site) - want) <= 1e-12 * max(1.0, abs(want))
