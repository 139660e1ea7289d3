"""Small functions of the device code, built for the host and checked over
their whole range."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host_harness")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CLANG = "/opt/rocm/llvm/bin/clang++"

pytestmark = pytest.mark.skipif(not (os.path.exists(HIPCC) and os.path.exists(CLANG) and os.path.exists(HERE)),
                                reason="no ROCm toolchain, or no host harness")


@pytest.fixture(scope="module")
def math(tmp_path_factory):
    d = str(tmp_path_factory.mktemp("math"))
    obj, so = os.path.join(d, "m.o"), os.path.join(d, "libdm.so")
    subprocess.run([HIPCC, "-c", "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2608_21920_amd", "csrc"),
                    os.path.join(HERE, "device_math.hip"), "-o", obj], check=True, capture_output=True)
    # (no kernel is launched: the runtime's symbols and the device code's stay without a value)
    und = subprocess.run(["nm", "-u", obj], check=True, capture_output=True, text=True).stdout
    syms = [w for w in und.split() if w.startswith(("__hip", "hip"))]
    subprocess.run([CLANG, "-shared", "-fPIC", obj, "-o", so, "-Wl,-Bsymbolic"] + ["-Wl,--defsym=%s=0" % s for s in syms
                   if s.startswith("__hip_fatbin")] + ["-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"],
                   check=True, capture_output=True)
    return so


def test_wrap_cell_of_boxes_shorter_than_the_margin(math):
    # every cell a particle can reach between re-sorts (64 cells past either
    # end of the box) and every node of a 256-cell window
    f = C.CDLL(math).dm_wrap_cell
    for n in list(range(2, 70)) + [127, 128, 129, 255, 1000]:
        for c in range(-64, n + 256):
            assert f(c, n) == c % n, (c, n)


def test_spectrum_bin_guess(math):
    # the momentum spectra's first guess is the true count of edges or one
    # beside it, and every edge lies below an infinite momentum
    f = C.CDLL(math).dm_spec_guess
    f.argtypes = [C.c_float]
    thr = np.array([10.0 ** (2.0 * (-2.0 + b / 8.0)) for b in range(89)])
    edges = np.sqrt(thr).astype(np.float32)
    p = np.concatenate([edges, np.nextafter(edges, np.float32(0)), np.nextafter(edges, np.float32(np.inf)),
                        np.geomspace(1e-2, 3.4e38, 20000).astype(np.float32)])
    p = p[p.astype(np.float64) ** 2 >= thr[0]]
    want = np.searchsorted(thr, p.astype(np.float64) ** 2, side="right")
    got = np.array([f(float(x)) for x in np.log2(p)])
    assert np.abs(got - want).max() <= 1 and got.min() >= 1 and got.max() == 89
    assert f(float("inf")) == 89 and f(-float("inf")) == 1
