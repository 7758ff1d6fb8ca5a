"""The sketch products around the tile total that decides whether they split
the contraction depth between wavefronts, against the oracle (tolerances of the
parity tests of the truncation: 1e-10 s_1, orthonormality 1e-12, chi' exact),
and an unsorted batch: problems are queued by size, results stay in place."""
import numpy as np
import pytest

import test_gpu_rrsvd as rr
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,m,n,chi_max", [(400, 32, 30, 6), (401, 32, 30, 6),
                                               (100, 60, 33, 6), (134, 30, 95, 6), (2, 17, 300, 30)])
def test_around_the_tile_total(count, m, n, chi_max):
    gen = wl.rng(count + n)
    a = [wl.known_spectrum(m, n, np.exp(-np.arange(min(m, n)) / 2.0), gen) for _ in range(3)]
    mats = [a[i % 3] for i in range(count)]
    res = rr._gpu(mats, chi_max, 5, 2, 1e-10)
    for i in (0, 1, count - 1):
        ou, os_, ovh, ochi, ow, ost = rr._oracle(mats[i], i, chi_max, 5, 2, 1e-10)
        U, S, VH, chi, w, st = (r[i] for r in res)
        assert chi == ochi
        assert np.max(np.abs(S[:ochi] - os_)) <= 1e-10 * os_[0]
        rec = (U[:, :ochi] * S[None, :ochi]) @ VH[:ochi]
        assert np.max(np.abs(rec - (ou * os_[None, :]) @ ovh)) <= 1e-10 * os_[0]


def test_an_unsorted_batch_keeps_its_places():
    gen = wl.rng(12)
    shapes = [(20, 30), (300, 200), (20, 30), (90, 100), (5, 7), (300, 200), (64, 400)]
    mats = [wl.known_spectrum(m, n, np.exp(-np.arange(min(m, n)) / 4.0), gen) for m, n in shapes]
    rr._compare(mats, rr._gpu(mats, 20, 10, 2, 1e-10), 20, 10, 2, 1e-10)


def test_a_sweep_of_unlike_bonds():
    # 16 chains whose front moves through: sweeps of 300 to 1000 tiles, whose
    # largest bonds at first have many times the average's, so that the verdict
    # changes on the way.  Chain 0 alone (few tiles, always split) gives the
    # same bonds and Schmidt values; the rank modes decide alike, bit for bit.
    import torch
    from paper_1504_00992_amd import api, models as pm
    dims, hb = pm.spin_boson(40, 6)
    runs = {}
    for chains, mode in ((16, 1), (16, 2), (1, 2)):
        dev = api.DeviceMPS.product_state(chains, dims, [0] * 40, 24)
        drv = api.TEBD(dev, hb, 0.1, 24, p=6, q=2, trunc_eps=1e-10, seed=11, adaptive=mode)
        for _ in range(20):
            drv.step()
        torch.cuda.synchronize()
        runs[chains, mode] = (dev.gamma.clone(), dev.lam.clone(), dev.chi.clone(), drv.ws.status.clone())
    for a, b in zip(runs[16, 1], runs[16, 2]):
        assert torch.equal(a, b)
    n = runs[1, 2][2].numel()
    assert torch.equal(runs[16, 2][2].flatten()[:n], runs[1, 2][2].flatten())
    assert int(runs[1, 2][2].max()) >= 8
    lam = runs[1, 2][1].flatten()
    assert float((runs[16, 2][1].flatten()[:lam.numel()] - lam).abs().max()) <= 1e-10
