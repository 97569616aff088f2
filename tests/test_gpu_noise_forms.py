"""The noise kernels' forms: four samples per thread (large draws whose rows
can be stored 16 bytes a lane), one sample per thread otherwise, and a batch's
calls dealt to slices.  Whatever the form the bits are the oracle's."""
import numpy as np
import pytest

import workloads as W

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


# K * ceil(T m / 4) around 2^20 calls: the first draw of each pair is the last
# of one sample per thread, the second the first of four; then odd row counts,
# and a row length that is no multiple of four (one sample per thread)
@pytest.mark.parametrize("K,T,m", [(4096, 255, 4), (4096, 256, 4), (65536, 31, 2), (65536, 32, 2),
                                   (65540, 33, 2), (131072, 11, 3), (65537, 40, 2)])
def test_noise_draw_sizes(mppi, oracle_lib, K, T, m):
    sigma = np.linspace(0.2, 1.3, m).astype(np.float32)
    g = _np(mppi.noise(11, 5, 2, K, T, m, sigma))
    o = oracle_lib.noise(11, 5, 2, K, T, m, sigma)
    assert np.array_equal(g.view(np.uint32), o.view(np.uint32))


@pytest.mark.parametrize("calls", [1, 2, 4])
@pytest.mark.parametrize("K", [32770, 32833, 32767])
def test_context_noise_four_samples(mppi, oracle_lib, K, calls):
    """Ragged sample counts over padded rows, a deviation per step, the mean
    sample, and nothing written past the last sample."""
    wl = W.c1(K=K, T=66)
    rng = np.random.default_rng(K)
    sig_t = (np.asarray(wl.sigma, np.float64)[None, :]
             * rng.uniform(0.5, 1.5, (wl.T, wl.m))).astype(np.float32)
    wl = wl.replace(sigma_t=sig_t, mean_sample=1)
    ctl = mppi.Controller(wl)
    ctl.set_tuning(noise_calls=calls)
    ctl.sample()
    eps = _np(ctl.noise())
    ctl.close()
    o = oracle_lib.workload_noise(wl)
    assert np.array_equal(eps.view(np.uint32), o.view(np.uint32))
    assert np.all(eps[:, :, 0] == 0)


@pytest.mark.parametrize("tile", [64, 128, 256])
@pytest.mark.parametrize("n", [1, 5])
def test_batch_noise_slices(mppi, oracle_lib, n, tile):
    insts = [wl.replace(K=(1, 255, 258, 515, 1021)[i], mean_sample=1)
             for i, wl in enumerate(W.c4(n_instances=n))]
    ctl = mppi.Controller(insts)
    ctl.set_tuning(batch_tile=tile)
    ctl.sample()
    eps = ctl.split(_np(ctl.noise()), 3)
    ctl.close()
    for i, wl in enumerate(insts):
        o = oracle_lib.workload_noise(wl)
        assert np.array_equal(eps[i].view(np.uint32), o.ravel().view(np.uint32)), i


# one launch's samples grouped for the XCDs or not: around both limits of the
# rule (2048 samples, 10 MiB of noise), ragged, with one iteration's noise drawn
# ahead by the launch before; T 257 has no time-parallel rollout
@pytest.mark.parametrize("K,T", [(2047, 40), (2048, 40), (2049, 40), (6553, 200), (6561, 200),
                                 (9000, 33), (300, 257)])
def test_grouped_rollouts(mppi, oracle_lib, K, T):
    wl = W.c2("circles", K=K, T=T, iters=1)
    a, b = mppi.Controller(wl), mppi.Controller(wl)
    a.iterate(3)
    for _ in range(3):
        b.sample()
        eps, word = _np(b.noise()), b.stats()["iteration"]
        b.rollout()
        b.update()
    o = oracle_lib.noise(wl.seed, word, wl.instance, K, T, wl.m, wl.sigma)
    assert np.array_equal(eps.view(np.uint32), o.view(np.uint32))
    for x, y in ((a.costs(), b.costs()), (a.controls(), b.controls())):
        assert np.array_equal(_np(x).view(np.uint32), _np(y).view(np.uint32))
    a.close()
    b.close()


@pytest.mark.parametrize("K,T", [(65536, 79), (65536, 80), (65530, 81)])
def test_wide_noise(mppi, oracle_lib, K, T):
    wl = W.c3(K=K, T=T)
    ctl = mppi.Controller(wl)
    ctl.sample()
    eps = _np(ctl.noise())
    ctl.close()
    o = oracle_lib.workload_noise(wl)
    assert np.array_equal(eps.view(np.uint32), o.view(np.uint32))
