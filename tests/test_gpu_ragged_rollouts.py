"""One lane per sample at sample counts that leave a wave or a workgroup ragged:
samples are independent, so the costs (and crash counts) are bit for bit the first
ones of a context with whole groups, and nothing is written past the last one."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

MODELS = {"quadrotor": lambda K: W.c3(K=K, T=9), "integrator": lambda K: W.c1(K=K, T=21),
          "circles": lambda K: W.c2("circles", K=K, T=30, iters=1)}


def _run(wl, block):
    import paper_2409_07563_amd as mppi
    ctl = mppi.Controller(wl, debug=wl.cx is not None, rollout="lane")
    ctl.set_tuning(rollout_block=block)
    ctl.sample()
    ctl.rollout()
    out = [ctl.costs().cpu().numpy().view(np.uint32)]
    if wl.cx is not None:
        out.append(ctl.crashes().cpu().numpy())
    ctl.iterate(2)  # the launch that also draws noise
    out.append(ctl.costs().cpu().numpy())
    ctl.close()
    return out


@pytest.mark.parametrize("block", [64, 256])
@pytest.mark.parametrize("model", sorted(MODELS))
@pytest.mark.parametrize("K", [1, 31, 33, 64, 257, 2049, 2111])
def test_costs_of_a_ragged_launch(model, K, block):
    whole = -(-K // 256) * 256
    a, b = _run(MODELS[model](K), block), _run(MODELS[model](whole), block)
    for x, y in zip(a[:-1], b[:-1]):
        assert np.array_equal(x, y[:K])
    assert np.all(np.isfinite(a[-1]))
