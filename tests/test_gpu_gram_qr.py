"""Gram-based QR at the edges of its size classes, against the oracle.

Truncated SVDs and bond updates whose sketches sit at the edges of the 16 x 16
tiles (l = 15, 16, 17, ...), of the wavefront's problems (l <= 16, 64 rows), of
the LDS the factor takes (l = 80) and of the tile queue (rows l^2 = 200000,
l = 8).  Tolerances: those of the parity tests of the truncation and of the
bond update (singular values and reconstructions 1e-10 s_1, orthonormality
1e-12, chi' and status exact).  They leave room for this QR: one Cholesky pass
whose scaled pivots stay above 1/4 is orthonormal to about
4 u sqrt(rows) l <= 2e-13 here (u = 1.1e-16, random-walk sums), and a second
pass follows where they do not.
"""
import numpy as np
import pytest

import test_gpu_rrsvd as rr
import test_gpu_tebd as tb
import workloads as wl
from paper_1504_00992_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,chi_max,p", [
    (64, 64, 1, 1), (17, 16, 5, 10), (64, 63, 6, 10), (65, 64, 6, 10), (64, 64, 7, 10),
    (300, 40, 22, 10), (129, 128, 23, 10), (200, 190, 38, 10), (83, 80, 39, 10),
    (84, 80, 39, 10), (75, 75, 63, 10), (76, 90, 64, 10), (3125, 30, 6, 2), (3126, 30, 6, 2), (8192, 24, 5, 2),
    (90, 300, 71, 10), (300, 257, 100, 10), (300, 280, 246, 10)])
def test_truncation_at_the_edges(m, n, chi_max, p):
    gen = wl.rng(m * 1000 + n + chi_max)
    s = np.exp(-np.arange(min(m, n)) / (chi_max / 6.0))
    a = wl.known_spectrum(m, n, s, gen)
    U, S, VH, chi, w, st = rr._gpu([a], chi_max, p, 2, 1e-10)
    # a graded first sketch may be refused by the Gram (only the report of that differs)
    rr._compare([a], (U, S, VH, chi, w, st & ~_lib.DEV_QR_FALLBACK), chi_max, p, 2, 1e-10)


@pytest.mark.parametrize("m,n,chi_max", [(60, 50, 40), (70, 68, 60), (75, 68, 60), (400, 300, 70)])
@pytest.mark.parametrize("decay", [0.1, 0.2, 0.25])
def test_second_pass_of_an_ill_conditioned_sketch(m, n, chi_max, decay):
    # no power iteration: the QR of A Omega (kappa 1e3 to 1e8) decides the span,
    # and one Cholesky pass of it is not orthonormal to rounding
    gen = wl.rng(m + int(100 * decay))
    a = wl.known_spectrum(m, n, np.exp(-decay * np.arange(min(m, n))), gen)
    U, S, VH, chi, w, st = rr._gpu([a], chi_max, 3, 0, 0.0)
    rr._compare([a], (U, S, VH, chi, w, st & ~_lib.DEV_QR_FALLBACK), chi_max, 3, 0, 0.0)


@pytest.mark.parametrize("q", [0, 1])
def test_flat_spectrum_and_a_mixed_batch(q):
    # well conditioned first sketches (kept whole by the Gram), sizes of every
    # route in one batch, with and without power iterations
    gen = wl.rng(77 + q)
    mats = [wl.known_spectrum(m, n, np.linspace(1, 0.5, min(m, n)), gen)
            for m, n in [(40, 30), (64, 64), (65, 17), (150, 140), (700, 90), (20, 3)]]
    mats.append(np.zeros((50, 40), dtype=np.complex128))
    rr._compare(mats, rr._gpu(mats, 30, 10, q, 1e-10), 30, 10, q, 1e-10)


@pytest.mark.parametrize("dims,chis,bond,chi_max,p", [
    ([2, 2, 2, 2], [1, 32, 40, 32, 1], 1, 6, 10),      # 64 rows, l = 16
    ([2, 2, 2, 2], [1, 33, 40, 32, 1], 1, 6, 10),      # 66 rows on one side
    ([2, 2, 2, 2], [1, 70, 80, 70, 1], 1, 70, 10),     # l = 80: the factor in LDS
    ([2, 2, 2, 2], [1, 70, 80, 75, 1], 1, 71, 10),     # l = 81: in global memory
    ([2, 2, 2, 2], [1, 100, 90, 100, 1], 1, 100, 10),  # l = 110
])
def test_bond_updates_at_the_edges(dims, chis, bond, chi_max, p):
    tb.test_bond_update_matches_oracle(dims, chis, bond, chi_max, p)


@pytest.mark.parametrize("n,chi_max", [(192, 50), (207, 34), (300, 50), (300, 2), (60, 4)])
def test_refused_sketches_reach_the_householder_class_of_their_size(n, chi_max):
    # a zero matrix: every Gram is refused.  Sizes on the tile queue in QR
    # classes 1, 2 and 3, and below it; beside them a matrix that is kept.
    gen = wl.rng(n)
    mats = [np.zeros((n, n), dtype=np.complex128),
            wl.known_spectrum(n, n, np.exp(-np.arange(n) / (chi_max / 6.0)), gen)]
    U, S, VH, chi, w, st = rr._gpu(mats, chi_max, 10, 2, 1e-10)
    large = _lib.tebd_size_class(0, n, chi_max + 10) >= 2
    assert bool(st[0] & _lib.DEV_QR_FALLBACK) == large
    rr._compare(mats, (U, S, VH, chi, w, st & ~_lib.DEV_QR_FALLBACK), chi_max, 10, 2, 1e-10)


@pytest.mark.parametrize("chi_m", [10, 100])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_first_sketch_of_a_large_bond(chi_m, mode):
    # 200 x 110 (QR class 3): of rank 40 at most (the attempt is refused, the
    # pivoted QR reveals the rank) and of full rank; a sweep reports neither
    import torch
    from oracle import philox, mps as omps
    from paper_1504_00992_amd import api
    assert _lib.tebd_size_class(0, 200, 110) == 3
    dims, chis = [2, 2, 2, 2], [1, 100, chi_m, 100, 1]
    gam, lam = tb._random_chain(dims, chis, 31)
    gate = wl.random_unitary(4, wl.rng(3))
    dev = api.DeviceMPS.from_host([(gam, lam)], dims, 100)
    prm = api._lib.params(100, 10, 2, 1e-10, 1e-14, 1504, 5, 0, mode)
    ws = api.BondWorkspace(dev, prm)
    api.tebd_bond_update(dev, 0, 1, torch.from_numpy(gate).cuda(), prm, ws)
    torch.cuda.synchronize()
    ref = omps.MPS(gam, lam)
    info = omps.bond_update(ref, 1, gate, 100, 1e-10, "rrsvd",
                            philox.gaussian_omega(200, 110, 1504, 1, 5), 2)
    g_gam, g_lam = dev.to_host(0)
    assert len(g_lam[1]) == info["chi"]
    assert np.max(np.abs(g_lam[1] - ref.lambdas[1])) < 1e-10
    assert not int(ws.status.view(-1)[1 if ws.status.numel() > 1 else 0]) & _lib.DEV_QR_FALLBACK


@pytest.mark.parametrize("m,n,chi_max", [(300, 280, 50), (260, 255, 54), (250, 255, 55), (300, 300, 71),
                                         (300, 310, 86), (320, 300, 87), (260, 270, 118)])
def test_widths_of_the_fp32_product_path(m, n, chi_max):
    # l = 60, 64, 65, 81, 96, 97, 128: the factor in registers and LDS, and beyond;
    # the bound stated for FP32 products (1e-5 of s_1)
    import torch
    from paper_1504_00992_amd import api
    gen = wl.rng(m + n)
    a = wl.known_spectrum(m, n, np.exp(-np.arange(min(m, n)) / 25.0), gen)
    U, S, VH, chi, w, st = api.rrsvd_truncate([torch.from_numpy(a).cuda()], chi_max, 10, 2, 1e-10,
                                              1504, 0, precision=1)
    torch.cuda.synchronize()
    ou, os_, ovh, ochi, ow, ost = rr._oracle(a, 0, chi_max, 10, 2, 1e-10)
    c = int(chi[0])
    assert c == ochi and not int(st[0]) & _lib.DEV_QR_FALLBACK
    s = S[0].cpu().numpy()[:c]
    u, vh = U[0].cpu().numpy()[:, :c], VH[0].cpu().numpy()[:c]
    assert np.max(np.abs(s - os_)) <= 1e-5 * os_[0]
    assert np.max(np.abs((u * s) @ vh - (ou * os_) @ ovh)) <= 1e-5 * os_[0]
    assert np.allclose(u.conj().T @ u, np.eye(c), atol=1e-12)
    assert np.allclose(vh @ vh.conj().T, np.eye(c), atol=1e-12)


@pytest.mark.parametrize("count", [256, 257])
def test_around_one_problem_per_cu(count):
    # a workgroup per problem up to 256, from there the small ones eight to a
    # workgroup: small, wide and refused (zero) sketches side by side
    gen = wl.rng(count)
    small = [wl.known_spectrum(30, 28, np.exp(-np.arange(28) / 2.0), gen) for _ in range(3)]
    mats = [small[i % 3] for i in range(count)]
    mats[5] = np.zeros((30, 28), dtype=np.complex128)
    mats[100] = wl.known_spectrum(150, 120, np.exp(-np.arange(120) / 5.0), gen)
    res = rr._gpu(mats, 6, 5, 2, 1e-10)
    assert not np.any(np.asarray(res[1][5]))
    for i in (0, 4, 6, 7, 8, 100, count - 1):
        ou, os_, ovh, ochi, ow, ost = rr._oracle(mats[i], i, 6, 5, 2, 1e-10)
        U, S, VH, chi, w, st = (r[i] for r in res)
        assert chi == ochi
        assert np.max(np.abs(S[:ochi] - os_)) <= 1e-10 * os_[0]
        rec = (U[:, :ochi] * S[None, :ochi]) @ VH[:ochi]
        assert np.max(np.abs(rec - (ou * os_[None, :]) @ ovh)) <= 1e-10 * os_[0]


def _graded(n, l, low, gen):
    """A matrix of rank 2 l whose first singular value is 1 and the others at most
    `low`, and a test matrix whose sketch has orthonormal columns that all
    contain the first singular vector: A^H Q then has columns almost parallel.
    Also its factors, and the smallest scaled pivot of that Gram matrix (the
    squared sine between a column and those before it, by Householder QR)."""
    s = np.concatenate([[1.0], low * np.linspace(1.0, 0.5, l - 1), low * np.linspace(0.1, 0.05, l)])
    u, v, w = (wl.haar_isometry(k, c, gen) for k, c in ((n, 2 * l), (n, 2 * l), (l, l)))
    a, omega = (u * s) @ v.conj().T, np.ascontiguousarray((v[:, :l] / s[:l]) @ w)
    b = a.conj().T @ np.linalg.qr(a @ omega)[0]
    pivot = np.min(np.abs(np.diag(np.linalg.qr(b)[1])) / np.linalg.norm(b, axis=0)) ** 2
    return a, omega, u, s, v, pivot


@pytest.mark.parametrize("low", [1e-2, 1e-7])
@pytest.mark.parametrize("n,q", [(300, 0), (300, 2), (400, 0), (400, 2), (600, 0), (600, 2)])
def test_a_refused_later_sketch_is_reported(n, q, low):
    # l = 20: by a workgroup in QR classes 1 and 2, on the tile queue in class 3.
    # Refused below a scaled pivot of 1e-10, and reported in classes 2 and 3
    # whichever route refuses.
    a, omega, u, s, v, pivot = _graded(n, 20, low, wl.rng(n + q))
    assert (pivot < 1e-12) == (low == 1e-7) and not 1e-12 < pivot < 1e-6
    st = rr._gpu([a], 12, 8, q, 0.0, omegas=[omega])[5]
    assert st[0] == (_lib.DEV_QR_FALLBACK if low == 1e-7 and _lib.tebd_size_class(0, n, 20) >= 2 else 0)


@pytest.mark.parametrize("low", [1e-3, 1e-4, 2e-5, 1e-7])
@pytest.mark.parametrize("n,q", [(300, 2), (400, 2), (600, 1), (600, 2)])
def test_later_sketches_near_the_refusal(n, q, low):
    # Kept down to a scaled pivot of 1e-10, else refused.  Against the exact truncation: a kept pass
    # of pivot d perturbs the basis by u / sqrt(d) <= 1e-11 in directions that A
    # weights with `low`, a Householder QR by u: both below 1e-13 of s_1.
    gen = wl.rng(n + q)
    a, omega, u, s, v, pivot = _graded(n, 20, low, gen)
    assert not 0.5e-10 < pivot < 2e-10
    U, S, VH, chi, w, st = rr._gpu([a], 12, 8, q, 0.0, omegas=[omega])
    report = pivot < 1e-10 and _lib.tebd_size_class(0, n, 20) >= 2
    assert chi[0] == 12 and st[0] == (_lib.DEV_QR_FALLBACK if report else 0)
    assert np.max(np.abs(S[0] - s[:12])) <= 1e-13
    assert np.max(np.abs((U[0] * S[0]) @ VH[0] - (u[:, :12] * s[:12]) @ v[:, :12].conj().T)) <= 1e-13
    assert np.allclose(U[0].conj().T @ U[0], np.eye(12), atol=1e-12)
    assert np.allclose(VH[0] @ VH[0].conj().T, np.eye(12), atol=1e-12)


@pytest.mark.parametrize("low", [1e-3, 1e-4, 2e-5, 1e-7])
@pytest.mark.parametrize("n", [300, 400, 600])
def test_factor_of_almost_parallel_columns(n, low):
    # no power iteration: the QR of B^H itself has the small pivots, kept in two
    # passes or refused.  Its factor R has B's singular values to a backward
    # error of some u s_1 either way: 1e-13 (the sketch's own error, u / low of
    # the test matrix, enters squared).
    gen = wl.rng(n)
    a, omega, u, s, v, pivot = _graded(n, 20, low, gen)
    assert not 0.5e-10 < pivot < 2e-10
    U, S, VH, chi, w, st = rr._gpu([a], 12, 8, 0, 0.0, omegas=[omega])
    report = pivot < 1e-10 and _lib.tebd_size_class(0, n, 20) >= 2
    assert chi[0] == 12 and st[0] == (_lib.DEV_QR_FALLBACK if report else 0)
    assert np.max(np.abs(S[0] - s[:12])) <= 1e-13
    assert np.allclose(U[0].conj().T @ U[0], np.eye(12), atol=1e-12)
    assert np.allclose(VH[0] @ VH[0].conj().T, np.eye(12), atol=1e-12)


@pytest.mark.parametrize("n,chi_max,p,decay", [(400, 12, 8, 0.4), (400, 2, 3, 2.0), (400, 70, 3, 0.1),
                                               (400, 70, 3, 0.15)])
def test_a_kept_sketch_of_one_pass_is_not_orthonormal(n, chi_max, p, decay):
    # as test_second_pass_of_an_ill_conditioned_sketch, but kept for sure: kappa of
    # A Omega is 1e4 to 1e6, and no refusal is reported (QR classes 2 and 3, by a
    # workgroup and on the tile queue), so that the second pass is what makes
    # the result orthonormal to 1e-12 (one pass: u kappa^2 >= 1e-8)
    assert _lib.tebd_size_class(0, n, chi_max + p) >= 2
    gen = wl.rng(int(100 * decay))
    a = wl.known_spectrum(n, n - 20, np.exp(-decay * np.arange(n - 20)), gen)
    res = rr._gpu([a], chi_max, p, 0, 0.0)
    assert not res[5][0] & _lib.DEV_QR_FALLBACK
    rr._compare([a], res, chi_max, p, 0, 0.0)


@pytest.mark.parametrize("adaptive", [0, 1, 2])
def test_no_launch_marks_the_routes_of_small_problems(adaptive):
    # the routes of a truncation are in its descriptors, and the second pass of an
    # FP32-product sweep needs them anew only where a sketch may be a large one
    import torch
    from test_gpu_fp32_products import _kernels
    from paper_1504_00992_amd import api, models as pm
    gen = wl.rng(5)
    mats = [torch.from_numpy(wl.known_spectrum(m, n, np.exp(-np.arange(min(m, n)) / 9.0), gen)).cuda()
            for m, n in ((1, 1), (40, 30), (400, 300))]
    dims, hb = pm.transverse_ising(8)
    dev = api.DeviceMPS.product_state(1, dims, [0] * 8, 16)
    drv = api.TEBD(dev, hb, 0.1, 16, p=4, q=1, trunc_eps=1e-10, seed=5, adaptive=adaptive, precision=1)
    launches = _kernels(lambda: (api.rrsvd_truncate(mats, 30, 10, 1, 1e-10), drv.step()))
    assert "k_chol_mark" not in launches


@pytest.mark.parametrize("rank", [3, 0])
@pytest.mark.parametrize("m,n,chi_max,p,tries", [(1, 1, 1, 0, False), (30, 28, 6, 2, False), (30, 28, 6, 3, True),
                                                 (30, 28, 10, 6, True), (2000, 40, 3, 1, True)])
def test_first_sketches_that_try_the_gram(m, n, chi_max, p, tries, rank):
    # more than eight columns, or size class 2: an attempt before the pivoted QR,
    # which takes what it refuses (rank 3); the four QRs of the power iterations and
    # that of B^H follow
    from test_gpu_fp32_products import _kernels
    gen = wl.rng(m + p)
    r = min(m, n, rank or n)
    a = wl.known_spectrum(m, n, np.exp(-np.arange(r) / 4.0), gen)
    out = []
    launches = _kernels(lambda: out.append(rr._gpu([a], chi_max, p, 2, 1e-10)))
    U, S, VH, chi, w, st = out[0]
    assert launches["k_gram_qr"] == 5 + tries
    rr._compare([a], (U, S, VH, chi, w, st & ~_lib.DEV_QR_FALLBACK), chi_max, p, 2, 1e-10)
