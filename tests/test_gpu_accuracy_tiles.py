"""The Accuracy Check's residual at the edges of its 16 x 16 tiles: bases of 15
to 30 columns, 20, 52 and 64 rows, 3 to 16 probes, with the tolerances of its
parity test (chi' and status exact, lambda and blocks 1e-10, weights 1e-12)."""
import pytest

import test_gpu_tebd as tb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chis,decay,p,chi_max", [
    ([1, 16, 14, 16, 1], 0.3, 16, 16), ([1, 13, 12, 16, 1], 0.5, 5, 16),
    ([1, 5, 13, 15, 1], 0.2, 3, 16), ([1, 16, 13, 16, 1], 0.1, 2, 16),
    ([1, 16, 1, 16, 1], 1.0, 15, 16), ([1, 1, 1, 1, 1], 1.0, 1, 4)])
def test_residual_at_the_tile_edges(chis, decay, p, chi_max):
    tb.test_accuracy_check_bond_update_matches_oracle(chis, decay, p, chi_max)
