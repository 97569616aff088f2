"""The MLP rollout's forms (one wave per 16-sample tile; the MLP over 2 or 4 waves
with the bicycle and the cost in waves of their own) compute the same thing with
the same operations: costs and controls are equal bit for bit, at horizons of one
and two steps, horizons around the noise ring of eight, sample counts that leave
a tile ragged, both integrators, costs, precisions and trigonometries, and with
every sampling option."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def _run(mppi, wl, block, accurate):
    c = mppi.Controller(wl, accurate_trig=accurate)
    c.set_tuning(rollout_block=block)
    c.iterate(2)
    out = [t.cpu().numpy().view(np.uint32) for t in (c.costs(), c.controls())]
    c.close()
    return out


def _options(wl):
    rng = np.random.Generator(np.random.PCG64(7))
    return wl.replace(is_beta=1, mean_sample=1, zero_frac=0.3, gamma=0.7,
                      sigma_t=(0.2 + rng.random((wl.T, 2))).astype(np.float32))


@pytest.mark.parametrize("H,K,T,kw", [
    (64, 16, 1, {}), (64, 1, 2, {}), (64, 37, 7, {}), (64, 300, 8, {}), (64, 4113, 9, {}),
    (32, 333, 17, {}), (32, 15, 1, {}),
    (64, 100, 12, dict(integrator="euler")), (32, 100, 12, dict(integrator="euler")),
    (64, 100, 11, dict(cost="quadratic")), (64, 250, 15, dict(options=True)),
    (64, 65, 10, dict(accurate=True)), (32, 65, 10, dict(accurate=True, integrator="euler")),
])
@pytest.mark.parametrize("bf16", [0, 1])
def test_tile_forms_bitwise(H, K, T, kw, bf16):
    import paper_2409_07563_amd as mppi
    wl = W.c5(K=K, T=T, hidden=H).replace(mlp_bf16=bf16, lam=20.0)
    kw = dict(kw)
    accurate, options = kw.pop("accurate", False), kw.pop("options", False)
    if kw.get("cost") == "quadratic":
        kw["ref"] = wl.ref[-1]
    wl = wl.replace(**kw)
    if options:
        wl = _options(wl)
    one = _run(mppi, wl, 64, accurate)
    for block in (128, 256) if H == 64 else (128,):
        for a, b in zip(one, _run(mppi, wl, block, accurate)):
            assert np.array_equal(a, b), f"block {block}"
