"""Both sides of the lines between the noise kernels' forms and between the orders
of the rollout's workgroups, and what the stores leave alone."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# 2^20 Philox calls are the first with four samples per thread: the draw before it
# and that draw; 80 MiB of noise the first with 1024 samples per workgroup
@pytest.mark.parametrize("K,T,m", [(65536, 30, 2), (65536, 31, 2), (65532, 32, 2),
                                   (104856, 100, 2), (104860, 100, 2)])
def test_lines_between_the_forms(oracle_lib, K, T, m):
    import paper_2409_07563_amd as mppi
    sigma = np.linspace(0.2, 1.3, m).astype(np.float32)
    g = mppi.noise(11, 5, 2, K, T, m, sigma).cpu().numpy()
    o = oracle_lib.noise(11, 5, 2, K, T, m, sigma)
    assert np.array_equal(g.view(np.uint32), o.view(np.uint32))


# one and four samples per thread, 1024 samples per workgroup; rows that cannot be
# stored 16 bytes a lane
@pytest.mark.parametrize("K,T,m,ldk", [(300, 7, 2, 320), (65533, 33, 2, 65536),
                                       (65535, 81, 4, 65600), (65535, 33, 2, 65537),
                                       (70001, 40, 2, 70016)])
def test_nothing_past_the_samples(oracle_lib, K, T, m, ldk):
    import ctypes as C
    import paper_2409_07563_amd as mppi
    sigma = np.zeros(8, np.float32)
    sigma[:m] = 0.5
    buf = torch.full((T * m + 1, ldk), -77.0, device="cuda")
    mppi._abi.check(mppi.lib().mppi_noise(3, 1, 2, K, T, m,
                                          sigma.ctypes.data_as(C.POINTER(C.c_float)),
                                          buf.data_ptr(), ldk,
                                          torch.cuda.current_stream().cuda_stream))
    got = buf.cpu().numpy()
    o = oracle_lib.noise(3, 1, 2, K, T, m, sigma[:m]).reshape(T * m, K)
    assert np.array_equal(got[:-1, :K].view(np.uint32), o.view(np.uint32))
    assert np.all(got[:-1, K:] == -77.0) and np.all(got[-1] == -77.0)


# workgroups ordered by sample groups or not: 11 and 12 groups (12 are filled up to
# 16), and 10 MiB of noise
@pytest.mark.parametrize("K,T", [(2048, 33), (2816, 33), (2817, 33), (6528, 200), (6529, 200)])
def test_lines_between_the_orders(oracle_lib, K, T):
    import paper_2409_07563_amd as mppi
    wl = W.c2("circles", K=K, T=T, iters=1)
    a, b = mppi.Controller(wl), mppi.Controller(wl)
    a.iterate(3)
    for _ in range(3):
        b.sample()
        eps, word = b.noise().cpu().numpy(), b.stats()["iteration"]
        b.rollout()
        b.update()
    o = oracle_lib.noise(wl.seed, word, wl.instance, K, T, wl.m, wl.sigma)
    assert np.array_equal(eps.view(np.uint32), o.view(np.uint32))
    for x, y in ((a.costs(), b.costs()), (a.controls(), b.controls())):
        assert torch.equal(x, y)
    a.close()
    b.close()
