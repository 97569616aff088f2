"""The MLP rollout at more than two 16-sample tiles per CU, where whole rounds of
four tiles per CU run one wave each and the rest may be split over waves: costs,
controls and gradients are bit for bit those of the forms alone."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def _wl(H, K, T, bf16, options=False):
    wl = W.c5(K=K, T=T, hidden=H).replace(mlp_bf16=bf16, lam=200.0)
    if options:
        rng = np.random.Generator(np.random.PCG64(7))
        wl = wl.replace(is_beta=1, mean_sample=1, zero_frac=0.3, gamma=0.7,
                        sigma_t=(0.2 + rng.random((wl.T, 2))).astype(np.float32))
    return wl


def _costs(wl, block=0):
    import paper_2409_07563_amd as mppi
    c = mppi.Controller(wl)
    if block:
        c.set_tuning(rollout_block=block)
    c.iterate(2)
    out = [t.cpu().numpy().view(np.uint32) for t in (c.costs(), c.controls())]
    c.close()
    return out


# a round and 7 tiles, a round and 2 or 3 per CU, almost a round, two rounds and one
@pytest.mark.parametrize("H,K", [(64, 8200), (64, 12300), (64, 16384), (64, 16489), (64, 24581),
                                 (64, 36871), (32, 12300), (32, 17001), (32, 33000), (16, 8197)])
@pytest.mark.parametrize("bf16", [0, 1])
def test_costs_of_the_default_form(H, K, bf16):
    wl = _wl(H, K, 5, bf16, options=K % 2 == 1)
    default = _costs(wl)
    for block in ((64, 128) if H == 64 else (64,)):
        for a, b in zip(default, _costs(wl, block)):
            assert np.array_equal(a, b), block
    if not wl.zero_frac:  # one iteration of fewer samples, all split
        import paper_2409_07563_amd as mppi
        out = []
        for k in (K, 4000):
            c = mppi.Controller(wl.replace(K=k))
            c.iterate(1)
            out.append(c.costs().cpu().numpy().view(np.uint32))
            c.close()
        assert np.array_equal(out[0][:4000], out[1])


@pytest.mark.parametrize("H,K", [(64, 16489), (32, 12301)])
@pytest.mark.parametrize("bf16", [0, 1])
def test_gradients_of_the_default_form(H, K, bf16):
    import paper_2409_07563_amd as mppi
    wl = _wl(H, K, 5, bf16)
    dU = torch.from_numpy(np.random.default_rng(K).normal(size=(5, 2)).astype(np.float32)).cuda()
    grads = []
    for block in (0, 64):
        c = mppi.Controller(wl, requires_grad=True, checkpoint_every=3)
        if block:
            c.set_tuning(rollout_block=block)
        c.iterate(1)
        grads.append([t.cpu() for t in (c.controls(), c.backward(dU), *c.backward_iters(dU))])
        c.close()
    for a, b in zip(*grads):
        assert torch.equal(a, b)
