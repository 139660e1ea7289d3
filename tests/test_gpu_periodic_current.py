"""The current of periodic tubes, summed per wave: sorted leptons, the tail
(pairs born since the last re-sort) and waves that hold several tubes."""
import sys

import numpy as np
import pytest

from paper_2608_21920_amd import Gap, workloads
from paper_2608_21920_amd import gap as G

from gpu_util import by_id, gpu_leptons_as_oracle

pytestmark = pytest.mark.gpu


def _cfg(cells, ppc, seed, **kw):
    return dict(workloads.TINY, n_cells=cells, ppc_init=ppc, seed=seed, flags=G.PERIODIC, h_gap_frac=2.0,
                cap_leptons=1 << 20, cap_photons=1 << 20, **kw)


def test_mixed_tubes_equal_single_tubes():
    # tails of three small tubes share waves: two periodic, one not; the
    # sums are integers, so each tube equals its single run bit for bit
    cfgs = [_cfg(200, 16, 1), dict(workloads.TINY, n_cells=200, cap_leptons=1 << 20, cap_photons=1 << 20), _cfg(130, 9, 2)]
    gb = Gap(cfgs)
    gb.step(160)
    for t, c in enumerate(cfgs):
        print("case: tube", t, flush=True)
        sys.stdout.flush()
        g = Gap(c)
        g.step(160)
        assert g.es() == gb.es(t)
        assert np.array_equal(g.field(), gb.field(t))
        A, B = by_id(gpu_leptons_as_oracle(g.leptons())), by_id(gpu_leptons_as_oracle(gb.leptons(t)))
        for k in ("cell", "xi", "u", "w", "id"):
            assert np.array_equal(A[k], B[k]), k
        g.close()
    assert gb.counts(0)["err"] == 0
    gb.close()
