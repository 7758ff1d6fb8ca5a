"""The small SVD at the edges of its size classes, against the oracle.

q = 0 and flat to steep spectra, so that the Jacobi iteration has from a few to
many rotations to do; widths l at the edges of the 16 lanes per pair, of the
padded rows and of the classes (32 / 64).  Tolerances: those of the parity
tests of the truncation (singular values and reconstructions 1e-10 s_1,
orthonormality 1e-12); the rotations here are exact to a few u = 1.1e-16
each, and a few hundred of them touch a column.
"""
import numpy as np
import pytest

import test_gpu_rrsvd as rr
import test_gpu_tebd as tb
import workloads as wl
from paper_1504_00992_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l", [1, 2, 3, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64])
@pytest.mark.parametrize("decay", [0.0, 0.2, 3.0])
def test_widths_of_the_pair_kernels(l, decay):
    gen = wl.rng(100 * l + int(10 * decay))
    p = min(l - 1, 3)
    n = l + 5
    mats = [wl.known_spectrum(n + 2, n, np.exp(-decay * np.arange(n)) * np.linspace(1, 0.7, n), gen),
            wl.known_spectrum(n, n + 7, np.exp(-decay * np.arange(n)) * np.linspace(1, 0.6, n), gen)]
    U, S, VH, chi, w, st = rr._gpu(mats, l - p, p, 0, 0.0)
    assert not np.any(st & ~_lib.DEV_QR_FALLBACK)
    rr._compare(mats, (U, S, VH, chi, w, st & ~_lib.DEV_QR_FALLBACK), l - p, p, 0, 0.0)


@pytest.mark.parametrize("l", [65, 69, 70, 72, 73, 80, 81, 128, 129, 200, 256])
@pytest.mark.parametrize("steep", [0.0, 4.0, 24.0])
def test_widths_of_the_block_rounds(l, steep):
    # one block of 8 columns more or less, an odd number of blocks, the
    # register classes (128); beside it a narrower problem of the same batch;
    # spectra down to e^-24, above the rank tolerance 1e-13 of the first QR
    decay = steep / l
    gen = wl.rng(100 * l + int(steep))
    n = l + 5
    mats = [wl.known_spectrum(n + 2, n, np.exp(-decay * np.arange(n)) * np.linspace(1, 0.7, n), gen),
            wl.known_spectrum(72, 90, np.exp(-decay * np.arange(72)) * np.linspace(1, 0.6, 72), gen),
            wl.known_spectrum(40, 30, np.exp(-decay * np.arange(30)) * np.linspace(1, 0.6, 30), gen)]
    U, S, VH, chi, w, st = rr._gpu(mats, l - 3, 3, 0, 0.0)
    assert not np.any(st & ~_lib.DEV_QR_FALLBACK)
    rr._compare(mats, (U, S, VH, chi, w, st & ~_lib.DEV_QR_FALLBACK), l - 3, 3, 0, 0.0)


def test_a_batch_of_more_pairs_than_workgroups():
    gen = wl.rng(9)
    mats = [wl.known_spectrum(90 + i % 5, 85, np.exp(-0.1 * np.arange(85)), gen) for i in range(260)]
    U, S, VH, chi, w, st = rr._gpu(mats, 70, 10, 0, 0.0)
    pick = [0, 1, 2, 130, 258, 259]
    for i in pick:
        ou, os_, ovh, ochi, ow, ost = rr._oracle(mats[i], i, 70, 10, 0, 0.0)
        assert np.max(np.abs(S[i][:ochi] - os_)) <= 1e-10 * os_[0]
        rec = (U[i][:, :ochi] * S[i][None, :ochi]) @ VH[i][:ochi]
        assert np.max(np.abs(rec - (ou * os_[None, :]) @ ovh)) <= 1e-10 * os_[0]


@pytest.mark.parametrize("chi,cap,chi_max", [(70, 90, 80), (75, 100, 66), (110, 130, 125)])
def test_rank_modes_agree_bitwise_beyond_64_columns(chi, cap, chi_max):
    # adaptive 1 (only enqueues: a workgroup per problem) and 2 (the host knows
    # the sizes: a launch per round) rotate in the same order
    import torch
    from paper_1504_00992_amd import api
    dims, chis = [2, 2, 2, 2], [1, chi, chi, chi, 1]
    gam, lam = tb._random_chain(dims, chis, 5)
    gate = torch.from_numpy(wl.random_unitary(4, wl.rng(3))).cuda()
    out = []
    for mode in (1, 2):
        dev = api.DeviceMPS.from_host([(gam, lam)], dims, cap)
        prm = api._lib.params(chi_max, 10, 2, 1e-10, 1e-14, 1504, 5, 0, mode)
        ws = api.BondWorkspace(dev, prm)
        api.tebd_bond_update(dev, 0, 1, gate, prm, ws)
        torch.cuda.synchronize()
        out.append((dev.gamma.clone(), dev.lam.clone(), dev.chi.clone(), ws.disc.clone()))
    assert int(out[0][2].max()) > 64
    for a, b in zip(*out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("l", [20, 60, 74, 128, 200])
def test_a_factor_that_overflowed(l):
    # finite entries of 1e200 and a test matrix of 1e-200: A Omega is harmless and
    # keeps its rank, A^H Q and every column of the factor are not finite.  Reported,
    # and the matrix before it keeps its bits.
    gen = wl.rng(l)
    n = l + 60
    a = wl.known_spectrum(n, n - 5, np.linspace(1.0, 0.5, n - 5), gen)
    omega = np.ascontiguousarray(wl.ginibre(n - 5, l, gen))
    alone = rr._gpu([a], l - 10, 10, 1, 1e-10, omegas=[omega])
    U, S, VH, chi, w, st = rr._gpu([a, a * 1e200], l - 10, 10, 1, 1e-10, omegas=[omega, omega * 1e-200])
    assert st[0] == alone[5][0] and st[1] & _lib.DEV_NONFINITE and 1 <= chi[1] <= l - 10
    for x, y in zip((U[0], S[0], VH[0]), (r[0] for r in alone[:3])):
        assert np.array_equal(x, y)
