"""The per-bin tail statistic against the oracle (bit for bit but for the mean's fp64 sum) where
its select can go wrong: token counts around what a workgroup keeps in registers (8192), ranks
on the first and last value and next to ties, all keys equal, keys that differ in the lowest
bit only, in the sign, or in the highest digit, and a digit that one key decides."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_08446_amd import sparrow as S

pytestmark = pytest.mark.gpu


def values(kind, T, rng):
    if kind == "equal":
        return np.full(T, 0.75, np.float32)
    if kind == "last bit":
        return (np.full(T, 0x3f400000, np.uint32) + rng.integers(0, 2, T, dtype=np.uint32)).view(np.float32)
    if kind == "signs":
        return rng.choice(np.array([-1.5, -0.0, 0.0, 2.0], np.float32), T)
    if kind == "spread":
        return np.exp(rng.uniform(-60, 60, T)).astype(np.float32) * rng.choice([-1, 1], T).astype(np.float32)
    return (1.0 - rng.beta(0.3, 4.0, T) * 0.7).astype(np.float32)


@pytest.mark.parametrize("T", [1, 2, 3, 255, 1024, 8191, 8192, 8193, 20001])
@pytest.mark.parametrize("kind", ["equal", "last bit", "signs", "spread", "rates"])
def test_tail_edges(gpu_device, T, kind):
    rng = np.random.default_rng(T)
    alpha = values(kind, T, rng)
    pos = rng.integers(-10, 300, T).astype(np.int32)
    for n_bins, pct in ((1, 0.0), (1, 5.0), (1, 100.0), (4, 37.5), (40, 99.0)):
        q, m, c = S.tail_stats(torch.from_numpy(alpha).cuda(), torch.from_numpy(pos).cuda(),
                               64, n_bins, pct)
        rq, rm, rc = oracle.tail_stats(alpha, pos, 64, n_bins, pct)
        np.testing.assert_array_equal(c.cpu().numpy(), rc)
        np.testing.assert_array_equal(q.cpu().numpy(), rq)
        ok = rc > 0
        # (another order of at most 20001 fp64 additions)
        size = np.abs(alpha.astype(np.float64)).max()
        np.testing.assert_allclose(m.cpu().numpy()[ok], rm[ok], rtol=0, atol=20001 * 2.0**-53 * size)


def test_more_tokens_than_32_bits_count(gpu_device):
    """One bin of 2^32 + 11 tokens (34 GB), all but five with one key: a digit's count does not
    fit 32 bits.  The keys differ in the lowest bit only, so one pass decides the rank."""
    T = 2 ** 32 + 11
    if torch.cuda.mem_get_info(gpu_device)[0] < 10 * T:
        pytest.skip("needs 40 GB of free device memory")
    low, high = np.array([0x3f400000, 0x3f400001], np.uint32).view(np.float32)
    alpha = torch.full((T,), float(high), dtype=torch.float32, device=gpu_device)
    alpha[:5] = float(low)
    pos = torch.zeros(T, dtype=torch.int32, device=gpu_device)
    torch.cuda.synchronize()
    q, m, c = (x.cpu().numpy() for x in S.tail_stats(alpha, pos, 64, 1, 50.0))
    assert c[0] == T
    assert q[0] == np.float64(high)
    assert low < m[0] <= high
    del alpha, pos
    torch.cuda.empty_cache()
