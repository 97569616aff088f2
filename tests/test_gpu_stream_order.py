"""Orders that the controller keeps by itself: eager calls against replays of a
graph that holds calls of the same controller.  Every result is bit for bit that
of the same calls made eagerly one after the other."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def test_eager_calls_between_replays():
    import paper_2409_07563_amd as mppi
    wls = W.c4(3, k_choices=(2000, 3333), t_choices=(40, 60))
    x0 = torch.as_tensor(np.concatenate([w.x0 for w in wls]), device="cuda")

    def call(ctl, x):
        ctl.set_state(x)
        ctl.shift(1)
        for _ in range(8):
            ctl.iterate(1)
        return ctl.controls()

    eager = mppi.Controller(wls)
    want = []
    call(eager, x0)
    for _ in range(5):
        call(eager, x0)
        eager.shift(2)
        eager.iterate(1)
        want.append(eager.controls().clone())
        eager.iterate(1)
    torch.cuda.synchronize()
    ctl = mppi.Controller(wls)
    call(ctl, x0)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(ctl, x0)
    got = []
    for _ in range(5):
        g.replay()
        ctl.shift(2)
        ctl.iterate(1)
        got.append(ctl.controls().clone())
        ctl.iterate(1)
    torch.cuda.synchronize()
    for i, (a, b) in enumerate(zip(got, want)):
        assert torch.equal(a, b), i
    ctl.close()
    eager.close()
