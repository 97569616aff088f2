"""Stand-alone draws of more samples than the contexts take, at the end of the
int32 range, in rows that can and cannot be stored 16 bytes a lane: the last
samples against the oracle's Philox words and Box-Muller tables."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [2**31 - 1024, 2**31 - 1023, 2**31 - 300, 2**31 - 4, 2**31 - 1])
def test_last_samples(oracle_lib, K):
    import torch
    import paper_2409_07563_amd as mppi
    if torch.cuda.mem_get_info()[0] < 12 << 30:
        pytest.skip("needs 12 GB of device memory")
    sigma = np.float32([0.7])
    seed, it, inst = 9, 4, 3
    eps = mppi.noise(seed, it, inst, K, 1, 1, sigma)
    ends = [(0, 4096), (K - 4096, K)]
    got = np.concatenate([eps[0, 0, a:b].cpu().numpy() for a, b in ends])
    del eps
    torch.cuda.empty_cache()
    k = np.concatenate([np.arange(a, b) for a, b in ends]).astype(np.uint32)
    ctr = np.stack([np.zeros_like(k), k, np.full_like(k, it), np.full_like(k, inst)], 1)
    x = oracle_lib.philox(ctr, [seed, 0])
    r, c, _ = oracle_lib.bm_tables()
    want = sigma[0] * (r[x[:, 0] >> 8] * c[x[:, 1] >> 8])
    assert np.array_equal(got.view(np.uint32), want.astype(np.float32).view(np.uint32))
