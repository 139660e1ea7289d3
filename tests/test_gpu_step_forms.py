"""That the handles whose two forms of a step are compared do take both."""
import pytest

from paper_2608_21920_amd import Gap, workloads

from test_gpu_fused_steps import CASES

pytestmark = pytest.mark.gpu

# form of the first step, and after the case's steps (2: in smaller pieces)
FORMS = {"tiny": (2, 2), "chunks": (1, 1), "least": (2, 2), "paper": (2, 2), "tubes": (2, 2)}


@pytest.mark.parametrize("name", list(CASES))
def test_compared_handles_take_both_forms(name):
    print("case:", name, flush=True)
    cfgs, steps = CASES[name]
    a, b = Gap(cfgs), Gap(cfgs)
    b.set_timing(True)
    got = []
    for n in (1, steps - 1, steps):
        a.step(n)
        b.step(n)
        got.append(a.step_form())
        assert b.step_form() == 0
    assert (got[0], got[2]) == FORMS[name], got
    a.set_timing(True)
    a.step(7)
    assert a.step_form() == 0
    a.close()
    b.close()


def test_captured_steps_are_fused():
    import torch
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        a = Gap(dict(workloads.TINY, rebucket_every=20), stream=s)
        for _ in range(4):
            a.step_graph(40)
            assert a.step_form() == 1
        a.close()


def test_a_window_s_steps_are_fused():
    g = Gap(dict(workloads.ADJOINT, n_cells=2000, ppc_init=8, cap_leptons=1 << 20, cap_photons=1 << 20))
    g.window_forward(20, 10)
    assert g.step_form() in (1, 2)
    g.backward()
    assert g.step_form() in (1, 2)
    g.close()
