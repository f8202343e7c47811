"""Lists that travel in the kernels' arguments (packs of up to 240 slots, blocks of up to 120) and the edge to lists on the device."""
import numpy as np
import pytest

from test_gpu_block import _check_single_block
from test_gpu_parity import _full_check
from test_gpu_plan_update import _Buffers

pytestmark = pytest.mark.gpu

SHORT = [1 + (i * 53) % 128 for i in range(31)]     # one tile each: with 8 heads, one slot per queue and sequence


@pytest.mark.parametrize("count", [1, 29, 30, 31])
@pytest.mark.parametrize("d", [64, 128])
def test_packed_lists_around_the_edge(count, d):
    import paper_2504_20490_amd as A
    lengths = SHORT[:count]
    for kind in (A.LIST_FWD, A.LIST_DKV):
        assert len(A.schedule(kind, A.build_cu_seqlens(lengths)[0], 8, 8)) == 8 * count
    _full_check(lengths, 8, 8, d, seed=400 + count + d, magnitude_slack=True, slack_roundings=2)


@pytest.mark.parametrize("count", [14, 15, 16])
def test_block_lists_around_the_edge(count):
    ql, kl = [130 - 7 * i for i in range(count)], [5 + 9 * i for i in range(count)]
    ql = [min(n, 128) for n in ql]
    kl = [min(n, 128) for n in kl]
    _check_single_block(ql, kl, [40 + i for i in range(count)], [3 * i for i in range(count)], 8, 8, 128, 500 + count,
                        f"block list of {8 * count} slots", magnitude_slack=True)


def test_refills_between_the_two_kinds_of_list():
    """Large, small, large, ...: each refill while the launches of the one before may still run."""
    import torch
    import paper_2504_20490_amd as A
    packs = [[5000, 3000, 1500], [17, 64, 111], [900, 7300, 33], [5], [4100, 1300, 800, 2500], [128] * 20, [2000, 129], [8000]]
    in_arguments = [False, True, False, True, False, True, True, False]
    bufs = [_Buffers(L, 4, 2, 128, 800 + i) for i, L in enumerate(packs)]
    longest = lambda plan: max(plan.num_items(kind) for kind in (A.LIST_FWD, A.LIST_DKV))
    fresh = []
    for b, short in zip(bufs, in_arguments):
        plan = A.Plan(A.build_cu_seqlens(b.lengths)[0], 4, 2, 128)
        assert (longest(plan) <= 240) == short, (b.lengths, longest(plan))
        b.launch(A, plan)
        torch.cuda.synchronize()
        fresh.append(b.results())
    for start in (1, 0):                                 # a plan that begins with a short list, and one that begins with a long one
        for b in bufs:
            for t in (b.o, b.lse, b.dq, b.dk, b.dv):
                t.fill_(float("nan"))
        torch.cuda.synchronize()
        plan = A.Plan(A.build_cu_seqlens(packs[start])[0], 4, 2, 128)
        for _ in range(2):
            for b in bufs:
                plan.update(A.build_cu_seqlens(b.lengths)[0])
                b.launch(A, plan)
        torch.cuda.synchronize()
        for b, want in zip(bufs, fresh):
            got = b.results()
            for n in got:
                assert np.array_equal(got[n], want[n]), (start, b.lengths, n)
