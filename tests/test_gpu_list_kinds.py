"""Work lists in the kernels' arguments and work lists in device memory are read by different instances of every attention kernel.
Both against the oracle, at every width that has kernels of its own, with whole items and with half items.  That these packs and
those of `test_gpu_whole_items.py` reach every instance is asked of the library on the CPU (`test_launched_kernels.py`)."""
import numpy as np
import pytest

import dispatch_packs as packs
from gpu_util import f64, make_case, to_dev
from oracle import rope as orope
from test_gpu_block import _check_single_block
from test_gpu_parity import _full_check
from test_gpu_rope import BASE, _assert_rounded, _bits, _table

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths,hq,hkv,d", packs.HALF_LONG_PACKS)
def test_half_items_with_lists_on_the_device(lengths, hq, hkv, d):
    run = _full_check(lengths, hq, hkv, d, seed=1900 + d + hq, magnitude_slack=True, ds_peak=True)
    assert run.plan.num_items(run.A.LIST_FWD) > 256          # two halves each: more than the forward has workgroups


@pytest.mark.parametrize("geometry,hq,hkv,d", packs.HALF_LONG_BLOCKS)
def test_half_items_of_blocks_with_lists_on_the_device(geometry, hq, hkv, d):
    run = _check_single_block(*geometry, hq, hkv, d, 2000 + d, f"half_long_block_d{d}", magnitude_slack=True)[0]
    assert all(run.plan.num_items(kind) > 120 for kind in (run.A.LIST_FWD, run.A.LIST_DKV))


@pytest.mark.parametrize("lengths,hq,hkv,d", packs.SHORT_PACKS)
def test_lists_in_the_arguments(lengths, hq, hkv, d):
    run = _full_check(lengths, hq, hkv, d, seed=2100 + d + hq, magnitude_slack=True, ds_peak=True)
    assert max(run.plan.num_items(kind) for kind in range(3)) <= 240


@pytest.mark.parametrize("geometry,hq,hkv,d", packs.SHORT_BLOCKS)
def test_lists_of_blocks_in_the_arguments(geometry, hq, hkv, d):
    run = _check_single_block(*geometry, hq, hkv, d, 2200 + d + hq, f"short_block_d{d}", magnitude_slack=True)[0]
    assert max(run.plan.num_items(kind) for kind in range(3)) <= 120


@pytest.mark.parametrize("hq,hkv,d", [(6, 2, 128), (6, 2, 104)])      # pieces of 16 bytes, of 8
@pytest.mark.parametrize("block", [False, True])
def test_rotation_with_lists_on_the_device(block, hq, hkv, d):
    """(The rotary tests' own packs have their lists in the arguments.)"""
    import torch
    import paper_2504_20490_amd as A
    ends = lambda lengths: np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    ql, kl, qp, kp = packs.HALF_GEOMETRY if block else (packs.HALF_LONG, packs.HALF_LONG, [0] * 38, [0] * 38)
    plan = A.BlockPlan(ends(ql), ends(kl), qp, kp, hq, hkv, d) if block else A.Plan(ends(ql), hq, hkv, d)
    assert max(plan.num_items(A.LIST_FWD), plan.num_items(A.LIST_DKV)) > (120 if block else 240)
    positions = max(p + n for ns, ps in ((ql, qp), (kl, kp)) for n, p in zip(ns, ps))
    for inverse in (False, True):
        q, k = make_case(ql, hq, hkv, d, seed=2300 + d)[0], make_case(kl, hq, hkv, d, seed=2400 + d)[1]
        qd, kd = to_dev(q), to_dev(k)
        qo, ko = torch.full_like(qd, float("nan")), torch.full_like(kd, float("nan"))
        A.rope_qk(plan, qd, kd, qo, ko, _table(positions, d), positions, inverse=inverse)
        torch.cuda.synchronize()
        turn = orope.rope_transposed if inverse else orope.rope
        for name, got, x, ns, ps in (("q", qo, q, ql, qp), ("k", ko, k, kl, kp)):
            pos = np.concatenate([p + np.arange(n) for n, p in zip(ns, ps)]).astype(np.int64)
            _assert_rounded(name, _bits(got), turn(f64(x), pos, BASE))
