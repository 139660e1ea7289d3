"""What libgap's host code asks of the HIP runtime, without a GPU: the library's
host side linked with a stand-in for the runtime (``host_harness/launches.cpp``)
that records launches, allocations and host copies.  No kernel runs."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2608_21920_amd import gap as G
from paper_2608_21920_amd import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host_harness")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CLANG = "/opt/rocm/llvm/bin/clang++"

pytestmark = pytest.mark.skipif(not (os.path.exists(HIPCC) and os.path.exists(CLANG) and os.path.exists(HERE)),
                                reason="no ROCm toolchain, or no host harness")


class Host:
    """The C ABI of a host-only build, with the recorder's questions."""

    def __init__(self, path):
        self.lib = lib = C.CDLL(path)
        for n, res, args in (("rec_stream", C.c_void_p, []), ("rec_count", C.c_longlong, []),
                             ("rec_name", C.c_char_p, [C.c_longlong]), ("rec_grid", C.c_longlong, [C.c_longlong]),
                             ("rec_allocs", C.c_longlong, []), ("rec_queued", C.c_longlong, []), ("rec_races", C.c_longlong, []),
                             ("rec_race", C.c_char_p, [C.c_longlong]),
                             ("rec_fail_at", None, [C.c_longlong]), ("rec_set_chunks", None, [C.c_longlong, C.c_longlong])):
            getattr(lib, n).restype, getattr(lib, n).argtypes = res, args
        lib.gap_init.argtypes = [C.c_void_p, C.c_int32, C.c_void_p, C.c_void_p, C.POINTER(C.c_void_p)]
        lib.gap_step.argtypes = lib.gap_step_graph.argtypes = [C.c_void_p, C.c_int64]
        lib.gap_sync.argtypes = lib.gap_free.argtypes = [C.c_void_p]
        lib.gap_diag.argtypes = [C.c_void_p, C.c_int32, C.c_int32, C.c_void_p, C.c_size_t, C.POINTER(C.c_size_t)]
        lib.gap_set_state.argtypes = [C.c_void_p, C.c_int32, C.c_int32, C.c_void_p, C.c_size_t]
        lib.gap_autotune.argtypes = [C.c_void_p, C.c_int32, C.c_void_p]
        self.stream = lib.rec_stream()

    def init(self, *cfgs):
        p = (G.GapParams * len(cfgs))(*[G.make_params(c) for c in cfgs])
        h = C.c_void_p()
        assert self.lib.gap_init(p, len(cfgs), self.stream, None, C.byref(h)) == 0
        return h

    def launches(self):
        """[(kernel, workgroups)] since the last call."""
        out = [(self.lib.rec_name(i).decode(), self.lib.rec_grid(i)) for i in range(self.lib.rec_count())]
        self.lib.rec_clear()
        return out

    def races(self):
        return [self.lib.rec_race(i).decode() for i in range(self.lib.rec_races())]


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = str(tmp_path_factory.mktemp("host"))
    obj, so = os.path.join(d, "gap.o"), os.path.join(d, "libgap_host.so")
    subprocess.run([HIPCC, "-c", "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC",
                    "-I" + os.path.join(ROOT, "include"), os.path.join(ROOT, "paper_2608_21920_amd", "csrc", "gap.hip"),
                    "-o", obj], check=True, capture_output=True)
    # (there is no device code: the symbol it would have stays without a value)
    und = subprocess.run(["nm", "-u", obj], check=True, capture_output=True, text=True).stdout
    fat = [w for w in und.split() if w.startswith("__hip_fatbin")]
    subprocess.run([CLANG, "-shared", "-fPIC", "-O1", "-std=c++17", "-Wno-unused-value", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", os.path.join(HERE, "launches.cpp"), obj, "-o", so, "-Wl,-Bsymbolic"]
                   + ["-Wl,--defsym=%s=0" % s for s in fat], check=True, capture_output=True)
    return Host(so)


def test_no_host_copy_runs_ahead_of_queued_fills(host):
    # a handle on a non-blocking stream, every kind of initial state and table
    for cfg in (workloads.TINY, dict(workloads.PAPER, n_cells=300, cap_leptons=1 << 16, cap_photons=1 << 16),
                dict(workloads.PRODUCTION, n_cells=300, cap_leptons=1 << 16, cap_photons=1 << 16)):
        h = host.init(dict(cfg, cap_leptons=1 << 16, cap_photons=1 << 16))
        assert host.lib.gap_step(h, 3) == 0
        host.lib.gap_free(h)
    assert host.races() == []


def _diag(host, h, kind, n):
    buf, wr = (C.c_char * max(n, 1))(), C.c_size_t(0)
    return host.lib.gap_diag(h, kind, 0, buf, n, C.byref(wr)), wr.value, bytes(buf)[:n]


@pytest.mark.parametrize("kind", [G.DIAG_COUNTS, G.DIAG_FIELD, G.DIAG_ES, G.DIAG_RHO, G.DIAG_NODE_E, G.DIAG_PROFILE,
                                  G.DIAG_PEAK, G.DIAG_SPECTRA, G.DIAG_PHASE, G.DIAG_ESPECTRUM, G.DIAG_DERIVED,
                                  G.DIAG_RETURN, G.DIAG_LEPTONS, G.DIAG_PROTONS, 99])
def test_a_refused_read_takes_notice_of_device_errors(host, kind):
    # a read that is refused (short buffer, unknown kind) waits like any
    # other: a device error comes before the refusal, and any other error
    # stops the run
    cfg = dict(workloads.TINY, n_cells=300, cap_leptons=1 << 14, cap_photons=1 << 14)
    for bits, want, after in ((8, -6, -6), (4, -1, -5), (0, -1, 0)):
        h = host.init(cfg)
        assert host.lib.gap_set_state(h, G.STATE_RAISE, 0, C.byref(C.c_int32(bits)), 4) == 0
        code, need, _ = _diag(host, h, kind, 1)
        if kind in (G.DIAG_LEPTONS, G.DIAG_PROTONS) and want == -1:
            assert code == 0 and need == 0       # (an empty store is not refused)
        else:
            assert code == want
        assert host.lib.gap_step(h, 1) == after
        host.lib.gap_free(h)


def test_a_read_that_fails_leaves_the_buffer_alone(host):
    h = host.init(dict(workloads.TINY, n_cells=300, cap_leptons=1 << 14, cap_photons=1 << 14))
    assert host.lib.gap_set_state(h, G.STATE_RAISE, 0, C.byref(C.c_int32(8)), 4) == 0
    buf, wr = (C.c_char * 1200)(*(b"x" * 1200)), C.c_size_t(0)
    assert host.lib.gap_diag(h, G.DIAG_FIELD, 0, buf, 1200, C.byref(wr)) == -6
    assert bytes(buf) == b"x" * 1200
    host.lib.gap_free(h)


def test_reading_particles_allocates_nothing(host):
    # (callers whose allocator is closed once a handle stands)
    cfg = dict(workloads.TINY, n_cells=300, cap_leptons=1 << 14, cap_photons=1 << 10)
    h = host.init(cfg)
    before = host.lib.rec_allocs()
    assert _diag(host, h, G.DIAG_LEPTONS, 0)[0] == 0
    assert _diag(host, h, G.DIAG_PHOTONS, 0)[0] == 0
    assert host.lib.rec_allocs() == before
    host.lib.gap_free(h)


def _chunky(host, lep, pho, **more):
    """A handle whose stores had `lep` and `pho` chunks at the last read."""
    h = host.init(dict(workloads.TINY, cap_leptons=1 << 16, cap_photons=1 << 16, **more))
    host.lib.rec_set_chunks(lep, pho)
    assert host.lib.gap_sync(h) == 0
    host.launches()
    return h


def _kernels(host, names=("k_sorted", "k_rest", "k_leptons", "k_photons", "k_tails", "k_pre")):
    """The particle kernels launched since the last call: (name, workgroups)."""
    return [(k, g) for n, g in host.launches() for k in names if k in n]


GENERAL = {"k_leptons", "k_photons", "k_tails", "k_pre"}
FUSED = {"k_sorted", "k_rest"}


def test_graph_replays_count_their_resorts(host):
    # 1024 cells are 8 tiles.  400 and 100 chunks: after a read a workgroup per
    # chunk (and 8 before them); once stores were re-sorted twice that many
    h = _chunky(host, 400, 100, rebucket_every=20)
    exact, loose = 8 + 400 + 104, 8 + 800 + 200
    step = lambda n: host.lib.gap_step(h, n)
    graph = lambda n: host.lib.gap_step_graph(h, n)
    assert step(1) == 0
    assert dict(_kernels(host))["k_sorted"] == exact
    assert step(19) == 0                           # the 20th step re-sorts
    host.launches()
    assert step(1) == 0
    assert dict(_kernels(host))["k_sorted"] == loose
    assert step(19) == 0
    # a replay of two re-sorts (capture and first replay in one call)
    assert graph(40) == 0
    assert host.lib.gap_sync(h) == 0
    host.launches()
    assert graph(40) == 0                          # a replay alone
    assert _kernels(host) == []
    assert step(1) == 0
    assert dict(_kernels(host))["k_sorted"] == loose
    assert step(19) == 0
    # three re-sorts since the last read: still the fused form; four: the general one
    assert host.lib.gap_sync(h) == 0
    assert step(20) == 0
    assert graph(40) == 0
    host.launches()
    assert step(1) == 0
    assert dict(_kernels(host))["k_sorted"] == loose
    assert step(19) == 0
    host.launches()
    assert step(1) == 0
    assert {k for k, _ in _kernels(host)} == GENERAL
    host.lib.gap_free(h)


def test_a_capture_and_its_replay_count_once(host):
    h = _chunky(host, 400, 100, rebucket_every=20)
    assert host.lib.gap_step_graph(h, 60) == 0     # three re-sorts, as many as the fused form is taken after
    host.launches()
    assert host.lib.gap_step(h, 1) == 0
    assert {k for k, _ in _kernels(host)} == FUSED
    host.lib.gap_free(h)


@pytest.mark.parametrize("pho,form", [(100, FUSED), (5000, GENERAL)])
def test_autotune_times_the_form_that_steps_take(host, pho, form):
    h = _chunky(host, 400, pho)
    chosen = (C.c_int32 * 4)()
    assert host.lib.gap_autotune(h, 4, chosen) == 0
    assert {k for k, _ in _kernels(host)} == form
    assert host.lib.gap_step(h, 2) == 0
    assert {k for k, _ in _kernels(host)} == form
    host.lib.gap_free(h)


def test_a_timed_handle_launches_each_pass_alone(host):
    h = _chunky(host, 400, 100)
    for on, form in ((1, GENERAL), (0, FUSED)):
        assert host.lib.gap_set_state(h, G.STATE_TIMING, 0, C.byref(C.c_int32(on)), 4) == 0
        assert host.lib.gap_step(h, 2) == 0
        assert {k for k, _ in _kernels(host)} == form
    host.lib.gap_free(h)


@pytest.mark.parametrize("lep", [100, 12287, 12288, 40000])
def test_the_launch_shape_read_is_the_one_launched(host, lep):
    # (a store of eight chunks per workgroup of a resident round takes two rounds)
    h = _chunky(host, lep, 5000)
    v, wr = (C.c_int32 * 4)(), C.c_size_t(0)
    assert host.lib.gap_diag(h, G.DIAG_LAUNCH, 0, v, 16, C.byref(wr)) == 0
    host.launches()
    assert host.lib.gap_step(h, 1) == 0
    ran = dict(_kernels(host))
    assert ran["k_leptons"] == v[0] and ran["k_photons"] == v[1]
    # written back, it is what the handle goes on with
    assert host.lib.gap_set_state(h, G.STATE_LAUNCH, 0, v, 16) == 0
    assert host.lib.gap_step(h, 1) == 0
    assert dict(_kernels(host)) == ran
    host.lib.gap_free(h)


@pytest.mark.parametrize("lep,pho,form", [(0, 0, 2), (255, 255, 2), (256, 0, 1), (0, 256, 1), (100000, 4096, 1),
                                          (0, 4097, 0), (-1, 0, 0)])
def test_the_form_of_a_step_by_the_sizes_last_read(host, lep, pho, form):
    h = _chunky(host, lep, pho)
    got = lambda: C.c_int32.from_buffer_copy(_diag(host, h, G.DIAG_FORM, 4)[2]).value
    assert host.lib.gap_step(h, 1) == 0
    assert got() == form
    assert {k for k, _ in _kernels(host)} == (FUSED if form else GENERAL)
    # captured steps take no smaller pieces: they are replayed on other counts
    assert host.lib.gap_step_graph(h, 1) == 0
    assert got() == min(form, 1)
    host.lib.gap_free(h)


@pytest.mark.parametrize("own_stream", [True, False])
def test_memory_is_given_back_after_the_work_that_uses_it(host, own_stream):
    # (an allocator may hand a block out again at once)
    hip = host.lib
    hip.hipMalloc.argtypes, hip.hipFree.argtypes = [C.POINTER(C.c_void_p), C.c_size_t], [C.c_void_p]
    left = []

    def alloc(n, ctx):
        p = C.c_void_p()
        assert hip.hipMalloc(C.byref(p), n) == 0
        return p.value

    def free(p, ctx):
        left.append(hip.rec_queued())
        hip.hipFree(p)
    al = G.GapAllocator(G.GapAllocator._fields_[0][1](alloc), G.GapAllocator._fields_[1][1](free), None)
    p = G.make_params(dict(workloads.TINY, cap_leptons=1 << 16, cap_photons=1 << 16, n_cells=300))
    h = C.c_void_p()
    assert hip.gap_init(C.byref(p), 1, host.stream if own_stream else None, C.byref(al), C.byref(h)) == 0
    assert hip.gap_step(h, 3) == 0
    assert hip.rec_queued() > 0
    hip.gap_free(h)
    assert left and set(left) == {0}


def test_a_failed_host_allocation_is_an_error_code(host):
    # (no exception crosses the C ABI: thrown through ctypes it would end this process)
    cfg = dict(workloads.PAPER, n_cells=3000, cap_leptons=1 << 16, cap_photons=1 << 16)
    h = host.init(cfg)
    g = C.c_void_p()
    p = (G.GapParams * 1)(G.make_params(cfg))
    buf = (C.c_char * (1 << 20))()
    part = (C.c_int64 * 2)(0, 0)
    try:
        host.lib.rec_fail_at(1000)
        for kind in (G.DIAG_FIELD, G.DIAG_RHO, G.DIAG_PROFILE, G.DIAG_SPECTRA, G.DIAG_ESPECTRUM):
            assert host.lib.gap_diag(h, kind, 0, buf, 1 << 20, None) == -2, kind
        assert host.lib.gap_init(p, 1, host.stream, None, C.byref(g)) == -2 and not g.value
        assert host.lib.gap_set_state(h, G.STATE_FIELD, 0, buf, 12008) == -2
        assert host.lib.gap_step(h, 2) == 0
    finally:
        host.lib.rec_fail_at(-1)
    # and the handle goes on
    assert host.lib.gap_diag(h, G.DIAG_FIELD, 0, buf, 1 << 20, None) == 0
    assert host.lib.gap_set_state(h, G.STATE_PARTICLES, 0, part, 16) == 0
    host.lib.gap_free(h)
