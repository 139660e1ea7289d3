"""Graph replays that contain re-sorts, then eager steps without a read between
(the stores have grown past the counts last read), against eager steps alone:
the same state bit for bit."""
import numpy as np
import pytest

from paper_2608_21920_amd import Gap, workloads

from test_gpu_fused_steps import _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("replays", [1, 2, 5])
def test_steps_after_unread_replays(replays):
    import torch
    print("case:", replays, "replays, then steps", flush=True)
    s = torch.cuda.Stream()
    cfg = dict(workloads.TINY, rebucket_every=20)
    a, b = Gap(cfg, stream=s), Gap(cfg, stream=s)
    b.set_timing(True)
    for g in (a, b):
        g.step(200)
        g.sync()
    for _ in range(3):
        for _ in range(replays):
            a.step_graph(40)
        a.step(13)
        a.step(7)
        b.step(40 * replays + 20)
        _same(a, b, 0)
    assert a.counts()["n_pho"] > 1000
    a.close()
    b.close()
