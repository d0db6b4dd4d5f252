"""The landmark build of large caches (the kernel that keeps a chunk's rows in LDS) against the
oracle, bit for bit.  The build is chosen by the block table's extent, so a wide block table
takes small caches there: chunks cut by the sequence's end at every remainder, odd head
counts (an odd number of rows in a burst), more heads than a workgroup holds, empty and
one-token sequences, absent pages."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_08446_amd import sparrow as S
from paper_2606_08446_amd import workloads as W

pytestmark = pytest.mark.gpu

WIDE = S.SPARROW_MAX_PAGES_PER_SEQ


@pytest.mark.parametrize("hkv,pages", [
    (8, (0, 1, 31, 32, 33, 64, 65, 200)), (3, (1, 63, 64, 65, 129, 2, 0, 300)),
    (5, (1, 50, 51, 52, 53, 103, 2, 7)), (300, (1, 2, 3, 0, 4, 1, 2, 5)),
])
def test_build_by_bursts(gpu_device, hkv, pages):
    ps = 16
    B = len(pages)
    assert hkv * ps * 256 * WIDE * B >= 1 << 30   # the build that this file is about
    rng = np.random.default_rng(hkv)
    lens = np.array([0 if p == 0 else ps * (p - 1) + int(rng.integers(1, ps + 1)) for p in pages],
                    np.int32)
    lens[1] = ps * (pages[1] - 1) + 1
    P = sum(pages) + 3
    perm = rng.permutation(P).astype(np.int32)
    bt = np.full((B, WIDE), -5, np.int32)
    at = 0
    for b, p in enumerate(pages):
        bt[b, :p] = perm[at:at + p]
        at += p
    absent = int(bt[-1, pages[-1] - 2])
    g = torch.Generator().manual_seed(hkv)
    k = torch.randn((P, hkv, ps, 128), generator=g).to(torch.bfloat16)
    k[0, 0, 0, :4] = torch.tensor([0.0, -0.0, 0.0, -0.0], dtype=torch.bfloat16)
    want = oracle.page_meta(W.bf16_bits(k), bt, lens)
    bt[-1, pages[-1] - 2] = P + 7                 # outside the cache: its row stays as it was
    want[absent] = 0
    meta = S.new_meta(P, hkv, gpu_device)
    S.page_meta_update(k.to(gpu_device), torch.from_numpy(bt).to(gpu_device),
                       torch.from_numpy(lens).to(gpu_device), meta)
    np.testing.assert_array_equal(W.bf16_bits(meta), want)
