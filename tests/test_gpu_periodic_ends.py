"""The node field at the ends of periodic tubes of one and several field
blocks: the average of the first and the last cell's field, bit for bit."""
import numpy as np
import pytest

from paper_2608_21920_amd import Gap, workloads
from paper_2608_21920_amd import gap as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [2, 3, 1000, 1023, 1024, 1025, 2048, 2049, 5000, 70001])
@pytest.mark.parametrize("more", [0, G.FILTER, G.FIELD_FROZEN])
def test_ends(cells, more):
    print("case:", cells, more, flush=True)
    if more == G.FILTER and cells < 16:
        return
    cfg = dict(workloads.BASE, n_cells=cells, init_kind=1, ppc_init=4, alpha=0.5, b=0.1, r_curv_cm=1e7, cap_leptons=1 << 20,
               cap_photons=1 << 12, flags=G.PERIODIC | G.QED_OFF | more)
    other = dict(cfg, n_cells=300, flags=G.QED_OFF)
    g = Gap([other, cfg])
    for n in (0, 1, 5):
        if n:
            g.step(n)
        E, node = g.field(1), g.node_field(1)
        assert node.size == cells + 1 and node[0] == node[-1]
        if more != G.FILTER:
            assert node[0] == np.float32(0.5) * (E[0] + E[-1])
        else:
            # the filter's node field is the average before rounding to FP32: three roundings of half an ulp
            assert abs(float(node[0]) - 0.5 * (float(E[0]) + float(E[-1]))) <= 1.5 * 2.0 ** -23 * max(abs(E[0]), abs(E[-1]))
    assert g.counts(1)["err"] == 0
    g.close()
