"""Periodic boxes shorter than the distance a particle covers between
re-sorts: it passes the box several times in its tile's window.  With a
re-sort after every step it never gets further than the next cell, and no
result depends on the interval: the same state bit for bit."""
import numpy as np
import pytest

from paper_2608_21920_amd import Gap, workloads
from paper_2608_21920_amd import gap as G

from gpu_util import by_id, gpu_leptons_as_oracle, gpu_photons_as_oracle

pytestmark = pytest.mark.gpu


def _state(n, seed):
    r = np.random.default_rng(seed)
    L = np.zeros(40 * n, G.LEPTON_DTYPE)
    L["cell"], L["frac"] = r.integers(0, n, L.size), r.integers(0, 1 << 24, L.size)
    L["u"] = (r.choice([-1, 1], L.size) * np.exp(r.uniform(0, 8, L.size))).astype(np.float32)
    L["w"] = np.where(np.arange(L.size) % 2, 1.0, -1.0)
    L["id"] = np.arange(L.size) + 1
    P = np.zeros(20 * n, G.PHOTON_DTYPE)
    P["cell"], P["frac"] = r.integers(0, n, P.size), r.integers(0, 1 << 24, P.size)
    P["x"] = (r.choice([-1, 1], P.size) * np.exp(r.uniform(1, 8, P.size))).astype(np.float32)
    P["w"], P["id"] = 1.0, np.arange(P.size) + 100001
    return L, P


@pytest.mark.parametrize("timed", [False, True])
@pytest.mark.parametrize("n", [2, 3, 30, 61, 62, 63, 64, 100])
def test_small_periodic_box_does_not_depend_on_the_resort(n, timed):
    print("case: periodic box of", n, "cells, timed", timed, flush=True)
    cfg = dict(workloads.TINY, n_cells=n, init_kind=2, flags=G.PERIODIC, h_gap_frac=2.0, cap_leptons=1 << 20,
               cap_photons=1 << 20)
    a, b = Gap(dict(cfg, rebucket_every=1)), Gap(cfg)
    for g in (a, b):
        g.set_timing(timed)                # (a timed handle takes the general form of the step)
        g.set_particles(*_state(n, n))
        g.step(150)
    ca, cb = a.counts(), b.counts()
    assert cb["rebuckets"] < ca["rebuckets"]
    for k in ("n_lep", "n_pho", "n_emit", "n_conv", "n_pho_exit", "err"):
        assert ca[k] == cb[k], k
    assert ca["n_emit"] > 0 and ca["err"] == 0
    assert a.es() == b.es()
    for f in ("field", "rho", "node_field", "spectra", "phase_space"):
        assert np.array_equal(getattr(a, f)(), getattr(b, f)()), f
    for A, B in ((by_id(gpu_leptons_as_oracle(a.leptons())), by_id(gpu_leptons_as_oracle(b.leptons()))),
                 (by_id(gpu_photons_as_oracle(a.photons())), by_id(gpu_photons_as_oracle(b.photons())))):
        for k in A:
            assert np.array_equal(A[k], B[k]), k
    a.close()
    b.close()
