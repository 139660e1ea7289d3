"""Particles saved and loaded, at the edges of the blocks and pieces in which
the device packs and unpacks their records."""
import ctypes as C

import numpy as np
import pytest

from paper_2608_21920_amd import Gap, workloads
from paper_2608_21920_amd import gap as G

pytestmark = pytest.mark.gpu


def _draw(n_lep, n_pho, cells):
    r = np.random.default_rng(n_lep + 7 * n_pho)
    L, P = np.zeros(n_lep, G.LEPTON_DTYPE), np.zeros(n_pho, G.PHOTON_DTYPE)
    for a in (L, P):
        a["cell"] = r.integers(0, cells, a.size)
        a["frac"] = r.integers(0, 1 << 24, a.size)
        a["id"] = r.permutation(a.size).astype(np.uint64) + np.uint64((1 << 40) + 1)
    L["u"], L["w"] = r.standard_normal(n_lep), r.choice([-1.0, 1.0, -2.5], n_lep)
    P["x"], P["w"], P["n0"] = r.choice([-1.0, 0.5, 3.0], n_pho), r.random(n_pho), r.integers(0, 1 << 20, n_pho)
    return L, P


def _sorted(a):
    return a[np.argsort(a["id"], kind="stable")]


# (with 1040 cells and up to 64 leptons a piece holds 9760 records)
@pytest.mark.parametrize("n_lep,n_pho", [(0, 0), (1, 0), (0, 1), (255, 257), (1023, 1025), (1024, 1024), (64, 9760), (64, 9761),
                                         (64, 30000), (50000, 20000)])
@pytest.mark.parametrize("periodic", [False, True])
def test_round_trip(n_lep, n_pho, periodic):
    print("case:", n_lep, n_pho, periodic, flush=True)
    g = Gap(dict(workloads.BASE, n_cells=1040, init_kind=2, alpha=0.0, b=0.1, r_curv_cm=1e7, cap_leptons=max(64, n_lep),
                 cap_photons=max(64, n_pho), flags=G.PERIODIC if periodic else 0))
    L, P = _draw(n_lep, n_pho, 1040)
    g.set_particles(L, P)
    gotL, gotP = g.leptons(), g.photons()
    assert _sorted(gotL).tobytes() == _sorted(L).tobytes()
    assert _sorted(gotP).tobytes() == _sorted(P).tobytes()
    assert g.leptons().tobytes() == gotL.tobytes() and g.photons().tobytes() == gotP.tobytes()
    c = g.counts()
    assert c["n_lep"] == n_lep and c["n_pho"] == n_pho
    g.close()


def test_a_refused_load_changes_nothing():
    g = Gap(dict(workloads.BASE, n_cells=1040, init_kind=2, alpha=0.0, b=0.1, r_curv_cm=1e7, cap_leptons=4096, cap_photons=4096))
    L, P = _draw(3000, 2000, 1040)
    g.set_particles(L, P)
    wantL, wantP = g.leptons().tobytes(), g.photons().tobytes()
    for species, name, value in ((0, "cell", 1040), (0, "cell", -1), (0, "frac", 1 << 24), (0, "w", 0.0), (1, "cell", 1040),
                                 (1, "frac", 1 << 24), (1, "x", 0.0)):
        bad = [L.copy(), P.copy()]
        bad[species][name][-1] = value
        with pytest.raises(G.GapError):
            g.set_particles(*bad)
        assert g.leptons().tobytes() == wantL and g.photons().tobytes() == wantP
    g.close()


def test_each_tube_of_an_ensemble_and_a_buffer_too_small():
    tubes = workloads.batched_qed_active(workloads.batched_tubes(3, seed=5))
    for c in tubes:
        c.update(n_cells=1040, ppc_init=3, cap_leptons=60000, cap_photons=60000)
    g = Gap(tubes)
    g.step(40)                                        # sorted slots and tails
    n = 0
    for t in range(3):
        L, P, c = g.leptons(t), g.photons(t), g.counts(t)
        assert L.size == c["n_lep"] and P.size == c["n_pho"]
        assert ((L["cell"] >= 0) & (L["cell"] < 1040) & (L["frac"] < 1 << 24) & (L["w"] != 0)).all()
        assert np.unique(L["id"]).size == L.size
        n += L.size
        buf, wr = np.full(L.nbytes, 7, np.uint8), C.c_size_t(0)
        code = g.lib.gap_diag(g.h, G.DIAG_LEPTONS, t, buf.ctypes.data, L.nbytes - 1, C.byref(wr))
        assert code == -1 and wr.value == L.nbytes and (buf == 7).all()
        assert g.lib.gap_diag(g.h, G.DIAG_LEPTONS, t, buf.ctypes.data, L.nbytes, C.byref(wr)) == 0
        assert buf.tobytes() == L.tobytes()
    assert n > 3 * 1040
    g.close()
