"""The controller's stream against the caller's: a tensor still being written on
torch's current stream (the default one or another) is read after it is ready,
what a call returns can be used there at once, and its memory is never handed
out while the library still works on it.  Every result is bit for bit that of
the same calls with the device synchronised in between."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def _slow(t, n=40):
    """t unchanged, after a few milliseconds of work on the current stream."""
    a = torch.ones((2048, 2048), device="cuda") / 2048
    for _ in range(n):
        a = a @ a
    return t * a[0, 0].round().clamp(1, 1)


def _loop(ctl, x0, wait, slow):
    out = []
    for i in range(4):
        x = x0 + 0.01 * i
        if slow:
            x = _slow(x)
        ctl.set_state(x)
        ctl.shift(1)
        ctl.iterate(2)
        if wait:
            torch.cuda.synchronize()
        U = ctl.controls()
        out.append((U * 2).clone())  # used at once on the current stream
        S = ctl.costs()
        out.append(S + 0)
        del U, S, x
        torch.full((ctl.T * ctl.m,), float("nan"), device="cuda")  # takes the freed memory
        if wait:
            torch.cuda.synchronize()
    return [t.cpu().numpy().view(np.uint32) for t in out]


@pytest.mark.parametrize("side", [False, True])
def test_order_with_the_callers_stream(side):
    import paper_2409_07563_amd as mppi
    wl = W.c2("circles", K=700, T=40, iters=1).replace(lam=20.0)
    x0 = torch.as_tensor(wl.x0, device="cuda")
    ref = mppi.Controller(wl)
    want = _loop(ref, x0, wait=True, slow=False)
    ref.close()
    s = torch.cuda.Stream() if side else torch.cuda.current_stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        ctl = mppi.Controller(wl)
        got = _loop(ctl, x0, wait=False, slow=True)
        ctl.close()
    for a, b in zip(want, got):
        assert np.array_equal(a, b)


def test_gradient_on_the_callers_stream():
    import paper_2409_07563_amd as mppi
    wl = W.c5(K=300, T=20, hidden=32).replace(lam=50.0)
    uref = torch.as_tensor(W.c5_uref(T=20), device="cuda")
    grads = []
    for slow in (False, True):
        ctl = mppi.Controller(wl, requires_grad=True)
        ctl.iterate(1)
        g = 2 * (ctl.controls() - uref)
        if slow:
            g = _slow(g)
        grads.append((ctl.backward(g) * 1).cpu())
        ctl.close()
    assert torch.equal(*grads)


def test_calls_join_a_capture_of_the_callers_stream():
    """A graph of one control call of a batch, captured from torch's current stream and
    replayed with eager work in between, gives what the eager calls give."""
    import paper_2409_07563_amd as mppi
    wls = W.c4(3, k_choices=(200, 333), t_choices=(20, 30))
    x0 = torch.as_tensor(np.concatenate([w.x0 for w in wls]), device="cuda")

    def call(ctl, x):
        ctl.set_state(x)
        ctl.shift(1)
        ctl.iterate(1)
        return ctl.controls()

    eager = mppi.Controller(wls)
    want = [call(eager, x0 + 0.1 * i).clone() for i in range(5)]
    ctl = mppi.Controller(wls)
    x = x0.clone()
    assert torch.equal(call(ctl, x), want[0])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        U = call(ctl, x)
    for i in range(1, 5):
        x.copy_(x0 + 0.1 * i)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(U, want[i]), f"replay {i}"
    ctl.close()
    eager.close()
