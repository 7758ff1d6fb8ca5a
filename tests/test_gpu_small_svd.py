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
