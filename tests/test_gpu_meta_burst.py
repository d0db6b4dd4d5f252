"""The landmark build of large caches (the kernel that keeps a chunk's rows in LDS) against the
oracle, bit for bit.  The build is chosen by the block table's extent, so a wide block table
takes small caches there.  The batch's pages are shared out evenly over the compute units:
workgroups without a page, with a few of several sequences, with several chunks; shares and chunks cut
by the sequences' ends, odd head counts (an odd number of rows in a burst), more heads than a
workgroup holds, empty and one-token sequences, absent pages, and the largest batch."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_08446_amd import sparrow as S
from paper_2606_08446_amd import workloads as W

pytestmark = pytest.mark.gpu

WIDE = S.SPARROW_MAX_PAGES_PER_SEQ


def check_build(device, hkv, pages, width):
    ps = 16
    B = len(pages)
    assert hkv * ps * 256 * width * B >= 1 << 30   # the build that this file is about
    rng = np.random.default_rng(hkv)
    lens = np.array([0 if p == 0 else ps * (p - 1) + int(rng.integers(1, ps + 1)) for p in pages],
                    np.int32)
    lens[1] = ps * (pages[1] - 1) + 1
    P = sum(pages) + 3
    perm = rng.permutation(P).astype(np.int32)
    bt = np.full((B, width), -5, np.int32)
    at = 0
    for b, p in enumerate(pages):
        bt[b, :p] = perm[at:at + p]
        at += p
    absent = int(bt[-1, pages[-1] - 2])
    g = torch.Generator(device=device).manual_seed(hkv)
    k = torch.randn((P, hkv, ps, 128), generator=g, device=device).to(torch.bfloat16)
    k[0, 0, 0, :4] = torch.tensor([0.0, -0.0, 0.0, -0.0], dtype=torch.bfloat16)
    want = oracle.page_meta(W.bf16_bits(k), bt, lens)
    bt[-1, pages[-1] - 2] = P + 7                 # outside the cache: its row stays as it was
    want[absent] = 0
    meta = S.new_meta(P, hkv, device)
    S.page_meta_update(k, torch.from_numpy(bt).to(device), torch.from_numpy(lens).to(device), meta)
    np.testing.assert_array_equal(W.bf16_bits(meta), want)


@pytest.mark.parametrize("hkv,pages", [
    (8, (0, 1, 31, 32, 33, 64, 65, 200)), (3, (1, 63, 64, 65, 129, 2, 0, 300)),
    (5, (1, 50, 51, 52, 53, 103, 2, 7)), (300, (1, 2, 3, 0, 4, 1, 2, 5)),
])
def test_build_by_bursts(gpu_device, hkv, pages):
    check_build(gpu_device, hkv, pages, WIDE)


@pytest.mark.parametrize("hkv,total,B", [(8, 9000, 41), (8, 16400, 7), (64, 1300, 20), (5, 13200, 4)])
def test_several_chunks_per_workgroup(gpu_device, hkv, total, B):
    """More pages than one chunk for every compute unit: 256 rows each of 256 units."""
    cus = torch.cuda.get_device_properties(gpu_device).multi_processor_count
    assert total > cus * min(64, 256 // hkv)
    cut = np.sort(np.random.default_rng(total).integers(0, total + 1, B - 1))
    pages = np.diff(np.concatenate(([0], cut, [total]))).tolist()
    pages[1], pages[-1] = max(1, pages[1]), max(2, pages[-1])
    check_build(gpu_device, hkv, [int(p) for p in pages], WIDE)


@pytest.mark.parametrize("B", [4096, 4097])
def test_largest_batch(gpu_device, B):
    """4096 sequences' page offsets fit beside the rows; more take the build page by page."""
    pages = np.random.default_rng(B).integers(0, 4, B)
    pages[1], pages[-1] = 3, 3
    check_build(gpu_device, 2, [int(p) for p in pages], 64)
