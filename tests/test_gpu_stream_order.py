"""Orders that the controller keeps by itself: eager calls against replays of a
graph that holds calls of the same controller, and the caller's next use of a
tensor's memory against the library's read of it.  Every result is bit for bit that
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


@pytest.mark.parametrize("reuse", ["freed", "overwritten", "binary64"])
def test_inputs_freed_or_overwritten_behind_a_long_queue(reuse):
    """set_state behind iterations still running, no tensor returned in between."""
    import paper_2409_07563_amd as mppi
    wl = W.c3(K=20000, T=100)
    base = torch.as_tensor(wl.x0, device="cuda")

    def states():
        return [base + 0.02 * i for i in range(5)]

    ref = mppi.Controller(wl)
    for x in states():
        ref.set_state(x)
        ref.iterate(4)
        torch.cuda.synchronize()
    want = ref.controls().clone()
    ref.close()
    ctl = mppi.Controller(wl)
    buf = torch.empty_like(base)
    torch.cuda.synchronize()
    for x in states():
        if reuse == "overwritten":
            buf.copy_(x)
            ctl.set_state(buf)
            buf.fill_(float("nan"))
        else:
            y = x * 1 if reuse == "freed" else x.double()
            n = y.numel()
            del x
            ctl.set_state(y)
            dtype = y.dtype
            del y
            junk = [torch.full((n,), float("nan"), dtype=dtype, device="cuda") for _ in range(8)]
            del junk
        ctl.iterate(4)
    got = ctl.controls().clone()
    torch.cuda.synchronize()
    ctl.close()
    assert torch.equal(got, want)
