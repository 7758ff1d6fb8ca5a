"""Truncated SVDs with complex FP32 products return the numbers they always
returned: the Gram-based QR between those products keeps one order and one
rounding of its sums (a last bit of Q that differs flips a rounding of 6e-8
here and there, which moves the truncated matrix by 1e-9 to 7e-8).

tests/golden/fp32_products.txt holds samples of results recorded from the
library's first version of that QR, column by column in LDS: per matrix the
largest singular values and entries of U diag(S) V^H x.  The inputs are exact
products, so that their bits do not depend on a BLAS.  Tolerance: 1e-12 of s_1;
the FP64 steps after the last FP32 product may round differently (about
1e-14), one flipped rounding is at least ten times the tolerance.
"""
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "fp32_products.txt")
KEPT = 8  # singular values, and as many entries of U diag(S) V^H x


def matrix(m, n, seed):
    """G diag(s) H of rank 212, s_i = 2^20 0.96^i: integers throughout, whose sums
    stay below 2^53, so that no order of a matrix product rounds."""
    gen = np.random.default_rng(seed)
    s = np.rint(2.0 ** 20 * np.cumprod(np.full(212, 0.96)))
    g, h = (gen.integers(-63, 64, shape) + 1j * gen.integers(-63, 64, shape)
            for shape in ((m, 212), (212, n)))
    return (g * s) @ h


def samples(mats, chi_max):
    import torch
    from paper_1504_00992_amd import api
    U, S, VH, chi, w, st = api.rrsvd_truncate([torch.from_numpy(a).cuda() for a in mats], chi_max, 10,
                                              2, 0.0, 1504, 0, precision=1)
    torch.cuda.synchronize()
    assert not st.cpu().numpy().any() and np.all(chi.cpu().numpy() == chi_max)
    out = []
    for i, a in enumerate(mats):
        m, n = a.shape
        u, s, vh = (t[i].cpu().numpy() for t in (U, S, VH))
        x = np.where(np.arange(n) % 3 == 0, 1.0, -0.5)
        y = (u[:, :chi_max] * s[:chi_max]) @ (vh[:chi_max] @ x) / np.sqrt(n)
        at = np.arange(KEPT) * 3
        out.append(np.concatenate([s[:KEPT], y[at].real, y[at].imag]))
    return out


def cases():
    """(m, n, chi_max, seed) and the recorded samples, line by line."""
    with open(GOLDEN) as f:
        for line in f:
            if not line.startswith("#"):
                w = line.split()
                yield tuple(int(v) for v in w[:4]), np.array([float.fromhex(v) for v in w[4:]])


@pytest.mark.parametrize("case,want", [pytest.param(c, w, id="-".join(map(str, c))) for c, w in cases()])
def test_results_of_fp32_products_stay(case, want):
    m, n, chi_max, seed = case
    got, = samples([matrix(m, n, seed)], chi_max)
    assert np.max(np.abs(got - want)) <= 1e-12 * want[0]


@pytest.mark.parametrize("chi_max", [50, 64, 86, 118])
def test_refused_sketches_of_fp32_products(chi_max):
    # l = 60, 74, 96 (the factor in LDS) and 128 (in global memory).  Only 20 rows
    # are not zero, so that the Gram of A Omega has rank 20 to FP64 rounding and
    # a pivot on the way is refused; a zero matrix, refused before the first
    # pivot; and between them one that is kept.  The bounds stated for FP32
    # products: 1e-5 of s_1, orthonormal to rounding.
    import torch
    import test_gpu_rrsvd as rr
    import workloads as wl
    from paper_1504_00992_amd import _lib, api
    gen = wl.rng(chi_max)
    thin = np.zeros((400, 400), dtype=np.complex128)
    thin[3::20] = wl.known_spectrum(20, 400, np.linspace(1.0, 0.1, 20), gen)
    mats = [thin, wl.known_spectrum(400, 380, np.exp(-np.arange(380) / 25.0), gen),
            np.zeros((380, 400), dtype=np.complex128)]
    assert _lib.tebd_size_class(0, 380, chi_max + 10) >= 2
    U, S, VH, chi, w, st = api.rrsvd_truncate([torch.from_numpy(a).cuda() for a in mats], chi_max, 10, 2,
                                              1e-10, rr.SEED, 0, precision=1)
    torch.cuda.synchronize()
    assert [bool(v & _lib.DEV_QR_FALLBACK) for v in st.cpu().numpy()] == [True, False, True]
    for i, a in enumerate(mats):
        ou, os_, ovh, ochi, ow, ost = rr._oracle(a, i, chi_max, 10, 2, 1e-10)
        c = int(chi[i])
        assert c == ochi
        u, s, vh = U[i].cpu().numpy()[:, :c], S[i].cpu().numpy()[:c], VH[i].cpu().numpy()[:c]
        assert np.max(np.abs(s - os_)) <= 1e-5 * os_[0]
        assert np.max(np.abs((u * s) @ vh - (ou * os_) @ ovh)) <= 1e-5 * os_[0]
        u = u[:, s > 0]
        assert np.allclose(u.conj().T @ u, np.eye(u.shape[1]), atol=1e-12)
        assert np.allclose(vh @ vh.conj().T, np.eye(c), atol=1e-12)


def _kernels(run):
    import torch
    from paper_1504_00992_amd import _lib
    torch.cuda.synchronize()
    _lib.tebd_profile_enable(True)
    try:
        run()
        torch.cuda.synchronize()
        return {k: v[1] for k, v in _lib.tebd_profile_read().items() if k.startswith("k_")}
    finally:
        _lib.tebd_profile_enable(False)


@pytest.mark.parametrize("m,n,rank,chi_max,p", [(30, 28, 4, 10, 6), (60, 60, 6, 16, 10), (96, 80, 10, 24, 10),
                                                (150, 140, 10, 38, 10), (400, 400, 10, 10, 10)])
def test_rank_deficient_matrices_with_fp32_products(m, n, rank, chi_max, p):
    # the FP32 rounding fills up the sketch, and the QR of B^H refuses the columns
    # beyond the rank: register classes (up to 150 x 140) are left to their
    # Householder kernel, which then runs the four QRs of the power iterations and this one
    import torch
    import test_gpu_rrsvd as rr
    import workloads as wl
    from paper_1504_00992_amd import _lib, api
    gen = wl.rng(m)
    a = wl.known_spectrum(m, n, np.linspace(1.0, 0.3, rank), gen)
    out = []
    launches = _kernels(lambda: out.extend(api.rrsvd_truncate([torch.from_numpy(a).cuda()], chi_max, p, 2, 1e-10,
                                                              rr.SEED, 0, precision=1)))
    cls = _lib.tebd_size_class(0, m, chi_max + p)
    if cls < 2:
        assert sum(v for k, v in launches.items() if k.startswith("k_qr_reg") and k.endswith("false>")) == 5
    U, S, VH, chi, w, st = out
    ou, os_, ovh, ochi, ow, ost = rr._oracle(a, 0, chi_max, p, 2, 1e-10)
    c = int(chi[0])
    assert c == ochi == rank and bool(int(st[0]) & _lib.DEV_QR_FALLBACK) == (cls >= 2)
    u, s, vh = U[0].cpu().numpy()[:, :c], S[0].cpu().numpy()[:c], VH[0].cpu().numpy()[:c]
    assert np.max(np.abs(s - os_)) <= 1e-5 * os_[0]
    assert np.max(np.abs((u * s) @ vh - (ou * os_) @ ovh)) <= 1e-5 * os_[0]
    assert np.allclose(u.conj().T @ u, np.eye(c), atol=1e-12)
    assert np.allclose(vh @ vh.conj().T, np.eye(c), atol=1e-12)


@pytest.mark.parametrize("mode", [0, 1, 2, 3])
def test_sweeps_with_fp32_products_use_no_gram_in_the_register_classes(mode):
    # their bonds are rank deficient while they grow
    from paper_1504_00992_amd import api, models as pm
    dims, hb = pm.spin_boson(12, 4)
    dev = api.DeviceMPS.product_state(2, dims, [0] * 12, 16)
    drv = api.TEBD(dev, hb, 0.1, 16, p=6, q=2, trunc_eps=1e-10, seed=5, adaptive=mode, precision=1)
    launches = _kernels(lambda: [drv.step() for _ in range(3)])
    assert not any(k.startswith("k_gram") for k in launches)
    assert int(drv.ws.status.max()) & ~(16 | 64 | 128) == 0
