"""How a pass deals out its items, beyond one workgroup per item.

Packs whose longest item outlasts the rest of a pass: the items are then shared out to two workgroups.  Parity with the
oracle where that split has its edges: a half without any key, a half of one key, one tile or an odd number of them per
head, groups of query heads (whose tiles follow one another in one item), head_dim below the tile width.  The
lists of these packs travel in the kernels' arguments; `test_gpu_list_kinds.py` has the same edges with lists on the device."""
import numpy as np
import pytest

import oracle
from dispatch_packs import EDGES   # (the longest decides that halves are taken)
from gpu_util import GpuRun, LSE_ABS, assert_close, default_scale, f64, make_case, magnitude_bound
from test_gpu_parity import _full_check

pytestmark = pytest.mark.gpu

MANY_SHORT = [1 + (i * 37) % 131 for i in range(40)] + [449] * 24


@pytest.mark.parametrize("hq,hkv,d", [(2, 2, 128), (3, 1, 128), (2, 1, 104), (4, 2, 64), (2, 2, 40)])
@pytest.mark.parametrize("lengths", [EDGES, [449], [700, 64], [1100]])
def test_items_shared_by_two_workgroups(lengths, hq, hkv, d):
    _full_check(lengths, hq, hkv, d, seed=900 + d + len(lengths), magnitude_slack=True)


@pytest.mark.parametrize("hq,hkv,d", [(8, 8, 128), (16, 8, 104), (8, 8, 72)])
def test_many_short_items(hq, hkv, d):
    """More than a thousand short dK/dV items: the pass then draws them in persistent workgroups, several per workgroup."""
    _full_check(MANY_SHORT, hq, hkv, d, seed=950 + d, magnitude_slack=True, slack_roundings=2)


@pytest.mark.parametrize("hq,hkv,d", [(2, 2, 128), (2, 1, 64), (2, 2, 96)])
@pytest.mark.parametrize("first", [1, 32])
def test_scores_below_the_range_of_fp32(first, hq, hkv, d):
    """Keys `first` .. `first` + 31 of every 64 have scores of about -6e38 before the scale, which fp32 holds as -inf: weight 0 in every row, as
    long as the row sees one other key.  The wave that owns the second half of every tile (first = 32) then meets no finite
    score at all."""
    lengths = [449, 70, 129]
    q, k, v, do = make_case(lengths, hq, hkv, d, seed=970 + d)
    to_bits = lambda x: np.uint16(np.float32(x).view(np.uint32) >> 16)
    position = np.concatenate([np.arange(n) for n in lengths])
    q[:, :, 0] = to_bits(2.0)
    k[(position % 64 >= first) & (position % 64 < first + 32), :, 0] = to_bits(-3e38)
    run = GpuRun(lengths, q, k, v, do).run()
    s = default_scale(d)
    ro, rlse = oracle.attn_fwd(f64(q), f64(k), f64(v), lengths, s)
    assert_close("O", run.host("o"), ro)
    assert np.max(np.abs(run.host("lse") - rlse)) <= LSE_ABS
    for name, ref in zip(("dq", "dk", "dv"), oracle.attn_bwd(f64(q), f64(k), f64(v), f64(do), lengths, s)):
        # column 0 of q is 2 in every row: column 0 of dK collects the bf16 roundings of dS times 2, where the bound is for N(0, 1)
        assert_close(name, run.host(name), ref, max_abs=(2 if name == "dk" else 1) * magnitude_bound(ref))
