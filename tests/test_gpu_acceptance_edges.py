"""The acceptance rate against the oracle at the edges of the kernel's layout: vocabularies
around what a thread keeps in LDS (9 vectors a row) and in registers (21 fp32 or 19 bf16 ones),
around whole groups of three of the rest, and around the one-wave kernel for short rows; more
tokens than workgroups (a workgroup's second token follows its first in the same registers),
with rows whose alignment changes from token to token; logits that exceed the first ones by
far, which move the sums' reference."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_08446_amd import sparrow as S

from parity import log

pytestmark = pytest.mark.gpu

# fp32 sums of up to 150000 terms over 512 threads and the exponents' rounding (2^-22 for terms
# up to 2^8 above the reference) stay under 2e-6.  The rounding of a log-sum-exp of base-2
# magnitude up to 64 is 2^-19; the two rows' roundings are made up for on average, so half
# their difference stays: at most 2^-19, a relative ln 2 x 2^-19.  With the jump the magnitude
# is 86 and the rounding 2^-18.
TOL = 2e-6
JUMP_TOL = TOL + np.log(2) * 2.0 ** -18


def rows(T, V, dtype, seed, jump):
    rng = np.random.default_rng(seed)
    a = (2 * rng.standard_normal((T, V))).astype(np.float32)
    b = a + (0.1 * rng.standard_normal((T, V))).astype(np.float32)
    if jump:                       # late entries far above everything before them
        at = rng.integers(V // 2, V, T)
        a[np.arange(T), at] += 60
        b[np.arange(T), at] += 55
    t = [torch.from_numpy(x).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
         for x in (a, b)]
    return t, [x.float().numpy() for x in t]


def check(T, V, dtype, seed, jump=False, tau=1.0):
    (a, b), host = rows(T, V, dtype, seed, jump)
    got = S.acceptance_rate(a.cuda(), b.cuda(), tau).cpu().numpy().astype(np.float64)
    want = oracle.acceptance(host[0], host[1], tau)
    tol = JUMP_TOL if jump else TOL
    assert np.abs(got - want).max() <= tol, np.abs(got - want).max()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("slots", [1, 9, 10, 12, 28, 29, 30, 31, 33, 34, 36])
@pytest.mark.parametrize("extra", [-1, 0, 1, 5])
def test_slot_edges(gpu_device, dtype, slots, extra):
    width = 4 if dtype == "f32" else 8
    check(3, slots * 512 * width + extra, dtype, slots + extra, jump=extra == 5)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V", [63, 64, 65, 71, 1000, 4099])
def test_several_tokens_per_workgroup(gpu_device, dtype, V):
    check(1100, V, dtype, V, tau=0.7)


@pytest.mark.parametrize("dtype,V", [("f32", 63001), ("bf16", 125003)])
def test_long_rows_several_tokens(gpu_device, dtype, V):
    check(300, V, dtype, V, jump=True, tau=-0.3 if dtype == "f32" else 1.0)


# One entry holds nearly all of the target's mass, and a vector of the others (w entries) adds
# less than half a unit of that entry's partial sum, so it is lost there: a chain of 24 vectors
# leaves the row's sum 24 w t short, t the others' size, and the rate here, the sum of the
# others under a flat draft row, is off by as much of itself.  (One chain of a thread's 122
# fp32 or 61 bf16 vectors: 6.3e-6, 3.1e-6.)  The partial sums and the sums over a wave and
# the workgroup add that entry to others 6 + 6 + 7 times, rounded to 2^-24 each.  The draft's
# values make its log-sum-exp nearly 0, with no rounding to share.
@pytest.mark.parametrize("dtype,value,flat,w", [("f32", -18.16, -12.4292, 4),
                                                ("bf16", -18.875, -12.4375, 8)])
def test_partial_sums_stay_short(gpu_device, dtype, value, flat, w):
    V, T = 250000, 40
    t = np.exp(value)
    assert w * t < 2.0 ** -24
    a = np.full((T, V), value, np.float32)
    at = np.linspace(0, V - 1, T).astype(np.int64)   # in LDS, in registers, read again
    a[np.arange(T), at] = 0
    b = np.full((T, V), flat, np.float32)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x, y = torch.from_numpy(a).to(dt), torch.from_numpy(b).to(dt)
    got = S.acceptance_rate(x.cuda(), y.cuda()).cpu().numpy().astype(np.float64)
    want = oracle.acceptance(x.float().numpy(), y.float().numpy(), 1.0)
    err = np.abs(got / want - 1)
    log(f"case partial sums {dtype}: {err.max():.2e}")
    assert err.max() <= 24 * w * t + 19 * 2.0 ** -24, err.max()
