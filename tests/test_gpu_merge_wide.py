"""Units whose lists are spread over many waves: the split of the list and the merge that takes
a workgroup per query head, against the oracle.

The sizes sit where the split's rules and the merge's loop change: one chunk or two per wave,
up to 64, 128 or 256 waves per unit, partials at the edges of a half-wave's share (8) and of a
round (128), and one unit, or 16 rows, more than the merge is used for; with units that one
wave held and sequences without pages among them, and one unit that nearly every wave (2000 of
them) has a part of."""
import pytest

from paper_2606_08446_amd import sparrow as S
from paper_2606_08446_amd import workloads as W

from parity import full_check, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group,hkv,ps,lengths", [
    (5, 1, 16, (1040,)), (2, 1, 16, (127 * 16,)), (2, 1, 16, (128 * 16 + 1,)),
    (2, 1, 16, (255 * 16 + 3,)), (4, 1, 16, (256 * 16,)), (8, 1, 16, (515 * 16,)),
    (16, 2, 16, (33000, 0)), (1, 3, 32, (2050, 70, 9000)), (3, 1, 128, (20000, 1, 129)),
    (2, 8, 16, (16, 4100)), (2, 8, 64, (900,) * 15 + (12000,)),
    (1, 3, 16, (1300, 0, 5) * 14 + (7000,)), (16, 3, 16, (700,) * 11),  # the half-wave merge
    (16, 2, 16, (2048,)), (11, 3, 16, (2048,)),   # 32 and 33 query-head rows: 128 and 64 waves
    (8, 2, 16, (1500, 2049)), (16, 1, 16, (4096, 4080)), (2, 1, 16, (16,) * 15 + (40000,)),
])
@pytest.mark.parametrize("out_dtype", [S.SPARROW_OUT_F32, S.SPARROW_OUT_BF16])
def test_spread_units(gpu_device, group, hkv, ps, lengths, out_dtype):
    log(f"case spread units: G={group} Hkv={hkv} ps={ps} lens={lengths} out={out_dtype}")
    w = W.small(B=len(lengths), Hq=group * hkv, Hkv=hkv, ps=ps, lengths=lengths, seed=len(lengths),
                schedule=W.fraction_budget(1, 2))
    full_check(W.generate(w, "cuda", lengths=list(lengths)), out_dtype=out_dtype)
