"""The rollout that a bicycle (RK4) context runs as created: the time-parallel
form with 16 or 32 lanes per sample, or the fused form, by the numbers of
samples and steps.  Whichever it is, the costs are bitwise those of the same
form chosen by hand, and follow the oracle."""
import numpy as np
import pytest

import workloads as W
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mppi():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2409_07563_amd as M
    M.lib()
    return M


def _np(t):
    import torch
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def _costs(ctl, wl):
    ctl.sample()
    ctl.rollout()
    return _np(ctl.costs()), _np(ctl.noise())


# both sides of every line: lanes of the time-parallel form, 0: fused
@pytest.mark.parametrize("K,T,lanes", [
    (1, 1, 32), (1024, 64, 32), (1025, 64, 16), (4096, 65, 32), (4097, 65, 16), (8192, 15, 16),
    (8193, 15, 0), (8193, 16, 16), (16385, 23, 0), (16385, 24, 16), (32769, 47, 0),
    (32769, 48, 16), (700, 256, 32), (700, 257, 0)])
@pytest.mark.parametrize("variant", ["circles", "costmap"])
def test_default_form(mppi, oracle_lib, variant, K, T, lanes):
    wl = W.c2(variant, K=K, T=T, iters=1)
    ctl = mppi.Controller(wl)
    assert ctl.tuning()["rollout_form"] == 0
    S, eps = _costs(ctl, wl)
    if lanes:
        ctl.set_tuning(rollout_form=2, lanes_per_sample=lanes, rollout_block=256)
    else:
        ctl.set_tuning(noise_calls=1)  # any setting selects what get_tuning reports
    S2, _ = _costs(ctl, wl)
    ctl.close()
    assert np.array_equal(S.view(np.uint32), S2.view(np.uint32))
    k = np.unique(np.linspace(0, K - 1, min(K, 600)).astype(int))
    sub = np.ascontiguousarray(eps[:, :, k])
    S_or, margin, _, slope = oracle_lib.rollout_costs(wl.replace(K=len(k)), eps=sub, slope=True)
    parity.assert_costs_close(S[k].astype(np.float64), S_or, margin, f"{variant} K{K} T{T}",
                              slope=slope if variant == "costmap" else None)


@pytest.mark.parametrize("kind", ["lane", "quad"])
def test_forced_forms_stay(mppi, kind):
    wl = W.c2("circles", K=500, T=60, iters=1)
    ctl = mppi.Controller(wl, rollout=kind)
    S, _ = _costs(ctl, wl)
    ctl.set_tuning(rollout_form=0, lanes_per_sample=1 if kind == "lane" else 4)
    S2, _ = _costs(ctl, wl)
    ctl.close()
    assert np.array_equal(S.view(np.uint32), S2.view(np.uint32))


def test_default_form_in_graphs(mppi):
    """Several iterations from one graph, replayed with other work between,
    equal the staged calls."""
    wl = W.c2("costmap", K=900, T=50, iters=1)
    a, b = mppi.Controller(wl), mppi.Controller(wl)
    for _ in range(3):
        a.iterate(2)
        for _ in range(2):
            b.sample()
            b.rollout()
            b.update()
        assert np.array_equal(_np(a.controls()).view(np.uint32), _np(b.controls()).view(np.uint32))
        assert np.array_equal(_np(a.costs()).view(np.uint32), _np(b.costs()).view(np.uint32))
    a.close()
    b.close()
