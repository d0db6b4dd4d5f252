"""Scoring and selection in one workgroup per unit against the split kernels, bit for bit.

Which of the two a call takes depends on its units and on the block table's width, so the
same sequences run both ways: all together behind a narrow table, and a few at a time behind a
wide one (the split kernels, which the oracle tests cover behind wide tables).  Page counts
sit at the edges of a wave's batch (16 pages), of a round over the waves (64 or 128), of a
block-table group (256 pages with four waves; eight waves' first group is the widest table) and of the
narrow tables themselves, with both workgroup sizes; with and without the append, both
landmarks, forced pages, more than eight query heads per KV head, absent pages in both groups,
lengths of 0 and past the table."""
import numpy as np
import pytest
import torch

from paper_2606_08446_amd import sparrow as S

from parity import one_workgroup_selection

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 2, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300, 511, 512, 271, 272,
         273, 319, 320, 321, 447, 448, 449]


def select(x, rows, width, append, landmark, sink, local, k_max):
    """(k, idx, meta, k_cache, v_cache) of the sequences `rows` behind a table of `width` pages;
    the caches are copies."""
    bt = torch.full((len(rows), width), 1 << 30, dtype=torch.int32, device="cuda")
    w = min(width, x["bt"].shape[1])
    bt[:, :w] = x["bt"][rows, :w]
    k, v, meta = x["k"].clone(), x["v"].clone(), x["meta"].clone()
    step = S.SparseDecodeStep(x["q"][rows].contiguous(), k, v, bt, x["lens"][rows].contiguous(),
                              meta, x["min"], x["num"], 100, 256, k_max, landmark=landmark,
                              sink_pages=sink, local_pages=local)
    stream = torch.cuda.current_stream().cuda_stream
    if append:
        step.append_score_topk(x["k_new"][rows].contiguous(), x["v_new"][rows].contiguous(),
                               stream)
    else:
        step.score_topk(stream)
    torch.cuda.synchronize()
    return step.k, step.idx, meta, k, v


@pytest.mark.parametrize("B,hkv,group,width", [
    (27, 2, 3, 448), (27, 3, 12, 448),    # few units, 512 threads
    (72, 2, 1, 512), (72, 2, 2, 480),     # 128 units and more
    (520, 1, 4, 512), (520, 1, 2, 449),   # 512 units and more: 256 threads
])
@pytest.mark.parametrize("append,landmark,sink,local", [
    (True, S.SPARROW_LANDMARK_MINMAX, 0, 0), (False, S.SPARROW_LANDMARK_MINMAX, 1, 3),
    (True, S.SPARROW_LANDMARK_MEAN, 2, 0), (False, S.SPARROW_LANDMARK_MEAN, 0, 0),
])
def test_paths_agree(gpu_device, B, hkv, group, width, append, landmark, sink, local):
    ps = 16
    rng = np.random.default_rng(width + hkv)
    assert one_workgroup_selection(B, hkv, width)
    pages = np.minimum(np.resize(EDGES, B), width)
    lens = np.where(pages > 0, (pages - 1) * ps + rng.integers(1, ps + 1, B), 0).astype(np.int32)
    P = int(pages.max()) * 2          # sequences share physical pages unless they append
    bt = np.stack([rng.permutation(P)[:512] for _ in range(B)]).astype(np.int32)
    P += B                            # a last page of its own for every sequence
    for b, n in enumerate(pages):
        if n:
            bt[b, n - 1] = P - B + b
    bt[3, 7] = P + 5                  # absent pages
    bt[9, 100] = -2
    bt[16, 300] = P + 9               # past the first block-table group of four waves
    lens[5] = width * ps + 40         # past the table: no append
    g = torch.Generator(device="cuda").manual_seed(width)

    def randn(*shape):
        return torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)

    x = dict(bt=torch.from_numpy(bt).cuda(), lens=torch.from_numpy(lens).cuda(),
             q=randn(B, hkv * group, 128), k=randn(P, hkv, ps, 128), v=randn(P, hkv, ps, 128),
             k_new=randn(B, hkv, 128), v_new=randn(B, hkv, 128),
             min=torch.full((40,), 3, dtype=torch.int32, device="cuda"),
             num=torch.arange(5, 45, dtype=torch.int32, device="cuda"))
    x["meta"] = S.new_meta(P, hkv, "cuda", landmark)
    S.page_meta_update(x["k"], torch.arange(P, dtype=torch.int32, device="cuda").view(P, 1),
                       torch.full((P,), ps, dtype=torch.int32, device="cuda"), x["meta"],
                       landmark=landmark)
    k_max = 200
    got = select(x, list(range(B)), width, append, landmark, sink, local, k_max)
    few = 36
    assert not one_workgroup_selection(few, hkv, 2100)
    for r0 in range(0, min(B, 180), few):
        rows = [r for r in range(r0, min(B, r0 + few)) if r != 5]
        want = select(x, rows, 2100, append, landmark, sink, local, k_max)
        assert torch.equal(got[0][rows], want[0])
        assert torch.equal(got[1][rows], want[1])
        for b in rows:
            if pages[b]:
                p = int(bt[b, pages[b] - 1])
                if 0 <= p < P:
                    for a, w in zip(got[2:], want[2:]):
                        assert torch.equal(a[p].view(torch.int16), w[p].view(torch.int16)), b
