"""Infinite momenta and energies, which a loaded state may hold, belong to the
overflow bins of the momentum spectra and of phase space."""
import numpy as np
import pytest

from paper_2608_21920_amd import Gap, workloads
from paper_2608_21920_amd import gap as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bin_cells", [1, 64])
def test_infinities_in_the_overflow_bins(bin_cells):
    print("case: infinite momenta, bins of", bin_cells, flush=True)
    g = Gap(dict(workloads.BASE, n_cells=200, init_kind=2, alpha=0.0, b=0.1, r_curv_cm=1e7))
    L, P = np.zeros(5, G.LEPTON_DTYPE), np.zeros(3, G.PHOTON_DTYPE)
    L["u"], L["w"], L["id"] = [np.inf, -np.inf, np.inf, 3e38, -3e38], [1, 1, -1, 1, -1], np.arange(5) + 1
    P["x"], P["w"], P["id"] = [np.inf, -np.inf, 3e38], 1, np.arange(3) + 11
    L["cell"], P["cell"] = 130, 131
    g.set_particles(L, P)
    g.set_profile_bin(bin_cells)
    s = g.spectra()
    assert s[:, 89].tolist() == [2.0, 3.0, 3.0] and s[:, :89].sum() == 0
    ph = g.phase_space()
    assert ph.sum() == 8
    assert ph[0, 130 // bin_cells, [0, 179]].tolist() == [1.0, 1.0]
    assert ph[1, 130 // bin_cells, [0, 179]].tolist() == [1.0, 2.0]
    assert ph[2, 131 // bin_cells, [0, 179]].tolist() == [1.0, 2.0]
    g.close()
