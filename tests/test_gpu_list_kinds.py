"""Work lists in the kernels' arguments and work lists in device memory are read by different instances of every attention kernel.
Both against the oracle, at every width that has kernels of its own, with whole items and with half items.  That these packs and
those of `test_gpu_whole_items.py` reach every instance is asked of the library on the CPU (`test_launched_kernels.py`)."""
import pytest

import dispatch_packs as packs
from test_gpu_block import _check_single_block
from test_gpu_parity import _full_check

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
