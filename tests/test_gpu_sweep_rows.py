"""The reverse sweep over more than 256 rows, where a workgroup holds two tiles (or
two units of the segment-parallel mode, of equal and unequal length), and over more
than a launch of rows: the gradient is bit for bit that of the one-wave sweep."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def _grads(wl, block, ckpt, tiles, iters):
    import paper_2409_07563_amd as mppi
    dU = np.random.default_rng(5).normal(size=(wl.T, 2)).astype(np.float32)
    c = mppi.Controller(wl, requires_grad=True, checkpoint_every=ckpt)
    c.set_tuning(rollout_block=block, adjoint_tiles=tiles)
    c.iterate(iters)
    out = [c.backward(torch.from_numpy(dU).cuda())] if iters == 1 else []
    out += c.backward_iters(torch.from_numpy(dU).cuda())
    assert float((c.weights() > 0).float().mean()) == 1.0 or iters > 1
    out = [t.cpu().numpy().view(np.uint32) for t in out]
    c.close()
    return out


def _same(wl, ckpt, tiles, iters=1):
    one = _grads(wl, 64, ckpt, tiles, iters)
    for block in (128, 256) if wl.mlp_hidden == 64 else (128,):
        for a, b in zip(one, _grads(wl, block, ckpt, tiles, iters)):
            assert np.array_equal(a, b), block


# 257 to 513 tiles: one workgroup with two, all of them, an odd one over
@pytest.mark.parametrize("H,K", [(32, 4097), (32, 4500), (64, 4500), (32, 8193), (64, 8200)])
@pytest.mark.parametrize("bf16", [0, 1])
def test_two_tiles_per_workgroup(H, K, bf16):
    _same(W.c5(K=K, T=7, hidden=H).replace(mlp_bf16=bf16, lam=300.0), ckpt=3, tiles=0)


@pytest.mark.parametrize("H", [32, 64])
def test_two_tiles_per_workgroup_through_two_updates(H):
    _same(W.c5(K=4200, T=6, hidden=H).replace(lam=300.0), ckpt=4, tiles=0, iters=2)


# checkpoints every 7 steps in units of 4 and 3; 23 steps leave a last segment of 2
@pytest.mark.parametrize("H", [32, 64])
@pytest.mark.parametrize("bf16", [0, 1])
@pytest.mark.parametrize("K,T,ckpt", [(2048, 23, 7), (1100, 23, 7), (1600, 33, 11)])
def test_units_of_unequal_length(H, bf16, K, T, ckpt):
    _same(W.c5(K=K, T=T, hidden=H).replace(mlp_bf16=bf16, lam=300.0), ckpt=ckpt, tiles=128)


@pytest.mark.parametrize("K", [32768, 33000, 49200])
def test_rows_in_several_launches(K):
    _same(W.c5(K=K, T=4, hidden=32).replace(lam=300.0), ckpt=2, tiles=0)
