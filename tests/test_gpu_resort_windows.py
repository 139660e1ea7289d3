"""Re-sorts around the tile counts where their LDS window changes: all tiles in
it, the most that fit, one more (a sliding window, the tails outside it), and
tubes that share a window.  No result depends on when the stores are sorted."""
import numpy as np
import pytest

from paper_2608_21920_amd import Gap, workloads

from gpu_util import by_id, gpu_leptons_as_oracle, gpu_photons_as_oracle

pytestmark = pytest.mark.gpu

QED = dict(workloads.TINY, ppc_init=2, u_init=2000.0, cap_leptons=4_000_000, cap_photons=4_000_000)


@pytest.mark.parametrize("cells", [[128], [128 * 1025], [128 * 2048], [128 * 2048 + 1], [128 * 1500, 128 * 700 + 5]])
def test_resort_interval_changes_no_result(cells):
    print("case: cells", cells, flush=True)
    a, b = (Gap([dict(QED, n_cells=n, seed=i, rebucket_every=r) for i, n in enumerate(cells)]) for r in (7, 40))
    a.step(45)
    b.step(45)
    for t in range(len(cells)):
        ca, cb = a.counts(t), b.counts(t)
        assert ca["err"] == 0 and ca["n_pho_born"] > 0
        for k in ("n_lep", "n_pho", "n_emit", "n_conv"):
            assert ca[k] == cb[k], k
        for ra, rb in ((gpu_leptons_as_oracle(a.leptons(t)), gpu_leptons_as_oracle(b.leptons(t))),
                       (gpu_photons_as_oracle(a.photons(t)), gpu_photons_as_oracle(b.photons(t)))):
            A, B = by_id(ra), by_id(rb)
            for k in A:
                assert np.array_equal(A[k], B[k]), k
        assert np.array_equal(a.field(t), b.field(t))
    a.close()
    b.close()
