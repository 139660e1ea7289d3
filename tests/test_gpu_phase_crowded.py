"""Phase space where many particles share a bin and a momentum column and go to
it without an LDS window: groups of one to many lanes of a wave in bins too
narrow for the LDS, and pairs in the tail.  The reference is a plain sum."""
import numpy as np
import pytest

from paper_2608_21920_amd import Gap, workloads
from paper_2608_21920_amd import gap as G

from test_gpu_diag_windows import _reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 8, 64])
def test_crowded_keys_equal_plain_sums(B):
    print("case: crowded phase space, bins of", B, flush=True)
    g = Gap(dict(workloads.TINY, init_kind=2, alpha=0.0, cap_leptons=1 << 20, cap_photons=1 << 20))
    # runs of 1, 2, ... 9 equal keys over and over, then whole waves of one key
    n = 4000
    run = np.repeat(np.arange(2000), np.arange(2000) % 9 + 1)[:n]
    L = np.zeros(2 * n, G.LEPTON_DTYPE)
    L["cell"] = np.concatenate([run % 1024, np.full(n, 300)])
    L["u"] = np.concatenate([10.0 ** (run % 7 - 2.0), np.full(n, -5.0)])
    L["w"] = np.concatenate([np.where(run % 3, 1.0, -2.0), np.full(n, 3.0)])
    L["id"] = np.arange(2 * n) + 1
    P = np.zeros(100000, G.PHOTON_DTYPE)
    P["cell"], P["frac"] = 500, np.random.default_rng(0).integers(0, 1 << 24, P.size)
    P["x"], P["w"], P["n0"], P["id"] = 1e6, 1.0, -3000, np.arange(P.size) + 100001
    g.set_particles(L, P)
    g.set_es_step(0.0, 0)
    g.set_profile_bin(B)
    for steps in (0, 1, 2):
        g.step(steps)
        prof, spec, phase = _reference(g, 0, B)
        assert np.array_equal(g.phase_space(), phase)
        assert np.array_equal(g.spectra(), spec)
    assert g.counts()["n_conv"] > 5000
    g.close()
