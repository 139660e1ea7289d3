"""Reads of the field and the charge around the size of the staging buffer, and
of the device's error word together with them."""
import numpy as np
import pytest

from paper_2608_21920_amd import Gap, workloads
from paper_2608_21920_amd import gap as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [2, 3, 524278, 524279, 524280, 1048559, 1048560, 1048561])
def test_field_and_charge_of_an_empty_gap(cells):
    print("case: cells", cells, flush=True)
    g = Gap(dict(workloads.BASE, n_cells=cells, init_kind=2, alpha=0.0, b=0.1, r_curv_cm=1e7, cap_leptons=1024, cap_photons=1024))
    # only the co-rotation background: E_{k+1/2} = dx (k + 1/2) in FP64, stored in FP32
    e = (0.25 / 16 / 2 ** 24) * (16 * 2 ** 24 * np.arange(cells, dtype=np.float64) + 8 * 2 ** 24)
    assert np.array_equal(g.field(), e.astype(np.float32))
    assert not g.rho().any()
    assert g.node_field()[-1] == np.float32(e[-1])
    # a charge in the last cell, half on each node
    L = np.zeros(1, G.LEPTON_DTYPE)
    L["cell"], L["frac"], L["w"], L["id"] = cells - 1, 1 << 23, 1.0, 1
    g.set_particles(L)
    rho = g.rho()
    assert rho[-1] == rho[-2] == 1 << 23 and not rho[:-2].any()
    g.close()


def test_error_word_comes_with_a_read():
    g = Gap(dict(workloads.TINY, n_cells=64))
    g.raise_device_error(4)
    assert g.field().size == 64                       # a read of data still gives it
    assert g.counts()["err"] == -5
    with pytest.raises(G.GapError):
        g.step(1)
    g.close()
