"""The spectrum of E at every number of stages: transforms of 2 to 2^17 cells,
of even and odd powers of two, padded and not."""
import numpy as np
import pytest

from paper_2608_21920_amd import Gap, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [2, 3, 4, 5, 8, 9, 16, 17, 33, 127, 256, 511, 1000, 2049, 4096, 4097, 16384, 100001])
def test_e_spectrum_against_numpy(cells):
    print("case: cells", cells, flush=True)
    g = Gap(dict(workloads.BASE, n_cells=cells, init_kind=2, alpha=0.0, b=0.1, r_curv_cm=1e7, cap_leptons=1024, cap_photons=1024))
    E = np.random.default_rng(cells).standard_normal(cells).astype(np.float32)
    g.set_field(E, 0.0)
    got = g.e_spectrum()
    M = 1
    while M < cells:
        M *= 2
    want = np.abs(np.fft.fft(E.astype(np.float64), M)[:M // 2 + 1]) ** 2 / M
    # |X_k| is off by at most a few eps log2(2 M) times the norm of the input, times sqrt(M) for one value
    eps = 4 * np.finfo(np.float64).eps * (1 + np.log2(M)) * np.sqrt(M) * np.linalg.norm(E.astype(np.float64))
    amp = np.sqrt(want * M)
    assert (np.abs(got - want) <= (2 * amp * eps + eps * eps) / M).all()
    g.close()
