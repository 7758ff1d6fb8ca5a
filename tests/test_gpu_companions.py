"""A result does not depend on what else is in the batch: the same bits alone,
beside a few matrices or chains and beside many (so that the launches take other
grids, tile variants and kernels' widths)."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


def _first(mats, chi_max, p, precision):
    import torch
    from paper_1504_00992_amd import api
    res = api.rrsvd_truncate(mats, chi_max, p, 2, 1e-10, 1504, 0, precision=precision)
    torch.cuda.synchronize()
    return [r[0].clone() for r in res]


def _matrix_among_others(m, n, chi_max, p, precision, others):
    # the matrix comes first, so that its test matrix is the same
    import torch
    gen = wl.rng(m)

    def mat(rows, cols):
        a = wl.known_spectrum(rows, cols, np.exp(-np.arange(min(rows, cols)) / 12.0), gen)
        return torch.from_numpy(a).cuda()
    a = mat(m, n)
    alone = _first([a], chi_max, p, precision)
    for rows, cols, count in others:
        for x, y in zip(alone, _first([a] + [mat(rows, cols)] * count, chi_max, p, precision)):
            assert torch.equal(x, y)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("m,n,chi_max,p", [(30, 28, 8, 6), (96, 80, 24, 10), (300, 400, 48, 10)])
def test_a_matrix_among_others(m, n, chi_max, p, precision):
    # fewer than the 400 tiles to which sketch products split their depth, and more
    _matrix_among_others(m, n, chi_max, p, precision,
                         [(28, 28, 300), (260, 250, 1), (260, 250, 70), (900, 800, 20)])


@pytest.mark.parametrize("mode", [0, 2, 3])
@pytest.mark.parametrize("model", ["tfim", "spin_boson"])
def test_a_chain_among_others(model, mode):
    # 16 chains whose bonds grow: sweeps of up to 1500 tiles of sketch products,
    # those of one chain stay below 100
    import torch
    from paper_1504_00992_amd import api, models as pm
    dims, hb = pm.transverse_ising(40) if model == "tfim" else pm.spin_boson(24, 8)
    state = []
    for chains in (1, 16):
        dev = api.DeviceMPS.product_state(chains, dims, [0] * len(dims), 32)
        drv = api.TEBD(dev, hb, 0.1, 32, p=6, q=2, trunc_eps=1e-12, seed=11, adaptive=mode)
        for _ in range(20):
            drv.step()
        torch.cuda.synchronize()
        state.append((dev.gamma[0].clone(), dev.lam[0].clone(), dev.chi[0].clone()))
    assert int(state[0][2].max()) >= 8
    for x, y in zip(*state):
        assert torch.equal(x, y)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("m,n,chi_max,p", [(80, 90, 100, 100), (140, 150, 60, 68), (500, 450, 64, 10),
                                           (70, 75, 190, 10)])
def test_a_wide_small_svd_among_others(m, n, chi_max, p, precision):
    # l = 80, 128, 74, 70, beside widths up to 200: the small SVD's kernels hold two
    # or four rows of a column per lane, by the widest problem
    _matrix_among_others(m, n, chi_max, p, precision, [(28, 28, 300), (260, 250, 1), (900, 800, 20)])


def test_tile_variants_give_the_same_bits():
    # the tuned variants of the sketch products (32 x 32, 64 x 64 and split-depth
    # 16 x 16 tiles), which are chosen by the largest matrix of a batch; depths
    # around the quarters' slabs of 16 and below one
    import torch
    from paper_1504_00992_amd import _lib, api
    gen = wl.rng(31)
    shapes = [(300, 200), (700, 650), (64, 65), (63, 128), (129, 17), (16, 15), (80, 49), (5, 3)]
    mats = [torch.from_numpy(wl.known_spectrum(m, n, np.exp(-np.arange(min(m, n)) / 9.0), gen)).cuda()
            for m, n in shapes]
    outs = []
    try:
        for v in (-1, 0, 1, 2):
            assert _lib.tebd_tune_set(0, 700, 74, v) == 0
            U, S, VH, chi, w, st = api.rrsvd_truncate(mats, 64, 10, 2, 1e-10, 1504, 0)
            torch.cuda.synchronize()
            outs.append([*U, *S, *VH, chi, w, st])
    finally:
        _lib.tebd_tune_set(0, 700, 74, -1)
    for o in outs[1:]:
        for x, y in zip(outs[0], o):
            assert torch.equal(x, y)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("m,n,chi_max,rank", [
    (190, 180, 24, 0), (190, 170, 38, 0), (192, 190, 54, 0), (260, 250, 20, 0), (300, 257, 20, 0),
    (320, 300, 20, 0), (321, 300, 20, 0), (384, 380, 22, 0), (96, 90, 80, 0), (190, 180, 24, 6), (300, 257, 20, 6)])
def test_a_register_class_sketch_on_and_off_the_tile_queue(m, n, chi_max, rank, precision):
    # alone and beside its like a workgroup takes it, beside a larger one the queue:
    # the same Gram matrix (one chunk of rows below 256, two from there on), factor,
    # second pass and Q
    import torch
    from test_gpu_fp32_products import _kernels
    gen = wl.rng(m + n)

    def mat(rows, cols, r):
        s = np.exp(-np.arange(r or min(rows, cols)) / 12.0)
        return torch.from_numpy(wl.known_spectrum(rows, cols, s, gen)).cuda()
    a, large = mat(m, n, rank), mat(700, 500, 0)
    out = []
    kernels = [_kernels(lambda: out.append(_first(x, chi_max, 10, precision)))
               for x in ([a], [a] * 5, [a, large], [a] + [large] * 7 + [a] * 3)]
    if precision == 0:
        on_queue = [any(k.startswith("k_chol<") for k in x) for x in kernels]
        assert on_queue == [m > 320, m > 320, True, True]
    for o in out[1:]:
        for x, y in zip(out[0], o):
            assert torch.equal(x, y)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("chi", [24, 60])
def test_rank_modes_agree_bitwise_where_a_sketch_may_be_large(chi, precision):
    # d = 8: bonds of 192 rows and l = 40 (register class 1, of the queue's size) and of
    # 480 rows and l = 85 (class 3); mode 1 knows the capacities, mode 2 the bonds.
    # Gates near the identity: sketches of full rank whose first stage is accepted.
    import test_gpu_tebd as tb
    import torch
    from paper_1504_00992_amd import _lib, api
    dims, chis, n = [8] * 6, [1, 8, chi, chi, chi, 8, 1], 6
    gam, lam = tb._random_chain(dims, chis, 41)
    g = []
    for b in range(n - 1):
        h = wl.ginibre(64, 64, wl.rng(b))
        ev, vec = np.linalg.eigh(h + h.conj().T)
        g.append((vec * np.exp(-0.01j * ev)) @ vec.conj().T)
    gates = torch.from_numpy(np.stack(g)).cuda()
    state = []
    for mode in (1, 2):
        dev = api.DeviceMPS.from_host([(gam, lam)], dims, 64)
        prm = _lib.params(64, 10, 1, 0.1, 1e-14, 1504, 3, precision, mode)
        ws = api.BondWorkspace(dev, prm)
        api.tebd_sweep(dev, gates, 0, prm, ws)
        torch.cuda.synchronize()
        assert not int(ws.status[0, 2]) & _lib.DEV_RANK_RETRY
        state.append((dev.gamma.clone(), dev.lam.clone(), dev.chi.clone(), ws.disc.clone(), ws.status.clone()))
    for x, y in zip(*state):
        assert torch.equal(x, y)
